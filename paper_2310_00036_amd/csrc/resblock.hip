// A whole IMPALA-ResNet residual block in one kernel (bf16 forward):
//
//   t = conv1(relu(x)) + b1,   y = x + conv2(relu(t)) + b2     (3x3 SAME convolutions, C -> C)
//
// Layer by layer the block moves five activation tensors through HBM (x for conv1; t, x and y
// for conv2; t written once); here it moves three (x read, t and y written). Each tile is a
// band of TH output rows of one frame:
//   - the input window, rows h0-2 .. h0+TH+1 of x, is staged HBM -> LDS (buffer loads, zero
//     padding from out-of-range offsets) and ReLU'd in place;
//   - conv1 computes t on the band's rows plus one halo row above and below (the halo rows
//     are recomputed by the neighbouring bands); t is rounded to bf16, the band's own rows
//     are stored (the backward pass reads them) and relu(t) goes to an LDS window with zero
//     padding columns, exactly what conv2 would have read from HBM;
//   - conv2 reads that window and writes y with the bias and the residual add fused; the
//     residual x comes from global memory into registers, fetched with the tile's staging.
// LDS layout (16 channels): each window is one plane, 32 bytes per pixel, pixels
// row-major with one zero padding column on each side. gfx950's LDS has 64 four-byte banks and
// serves a 16-byte read of a wave in four passes of 16 lanes (the lanes of each half-wave whose
// bits 2..4 have one parity); a pass is conflict-free when its 16 reads land on distinct 16-byte
// bank groups. A B fragment (lane (g, r): 8 k-values of pixel r) then spreads every pass over all
// 64 banks for any run of 16 consecutive window pixels, so a column tile is 16 consecutive window
// pixels, padding columns included (their outputs are dropped) and never a wrapped run of
// frame pixels, whose two-pixel jump at a row end would fold two reads onto one bank group.
// Per MFMA: 16 output pixels per column tile, one 16-byte B fragment per lane and k-step; the
// k-steps past the 9 taps read a zeroed 16-byte word. (32 channels: resblock_walk_fwd_kernel.)
// Each wave owns one 16-channel block of the outputs and holds both convolutions' A
// fragments for it in registers, loaded once per workgroup, so LDS holds only the windows.
#include "common.h"
#include "kernels.h"
#include "walk.h"

#include <algorithm>

namespace cb {

template <int C>
struct RbGeom {
    static constexpr int K = 9 * C;
    static constexpr int KSTEPS = (K + 31) / 32;
    static constexpr int MT = C / 16;                      // 16-channel planes (and output blocks)
    static constexpr int PXB = 32;                         // bytes per pixel and plane
    static_assert(C == 16, "32 channels have a kernel of their own");
    // Both weight sets in 8-wave workgroups at 4 waves per SIMD (128 registers).
    static constexpr int NW = 8;
    static constexpr int WPS = 4;                          // waves per SIMD (register budget)
    static constexpr int WGS = WPS * 4 / NW;               // workgroups per CU
    static constexpr int MAXS = 5;                         // x-window staging slots per lane
    static constexpr int MAXT = 5;   // conv2 column tiles per wave, whose residuals are fetched at the tile's start
    __host__ __device__ static int blocks(int slots) { return (slots + 63) / 64; }
    // x window: MT planes of (TH+4) x (W+2) pixels, in whole 1 KB staging blocks
    __host__ __device__ static int xwin_bytes(int TH, int W) { return blocks(MT * (TH + 4) * (W + 2) * 2) * 1024; }
    // relu(t) window: MT planes of (TH+2) x (W+2) pixels, then a zeroed 32-byte word
    __host__ __device__ static int twin_bytes(int TH, int W) { return MT * (TH + 2) * (W + 2) * PXB + 32; }
};

struct RbTile {
    int TH, nbands, ntiles;
    int x_off, t_off;   // LDS byte offsets of the two windows
    float inv_W, inv_TW;
};

template <int C, int NW>
__global__ __launch_bounds__(64 * NW, RbGeom<C>::WPS) void resblock_fwd_kernel(ResBlockArgs a, RbTile t) {
    using G = RbGeom<C>;
    constexpr int NT = 64 * NW, KSTEPS = G::KSTEPS, MT = G::MT, PXB = G::PXB;
    static_assert(NW % MT == 0, "waves split evenly over the output channel blocks");

    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* xw = smem + t.x_off;   // relu(x) window, MT planes of [TH+4][W+2] pixels
    unsigned char* tw = smem + t.t_off;   // relu(t) window, MT planes of [TH+2][W+2] pixels

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, r16 = lane & 15;
    const int H = a.H, W = a.W, TH = t.TH, TW = W + 2;
    const int xps = (TH + 4) * TW * PXB, tps = (TH + 2) * TW * PXB;   // plane strides (bytes)
    const int mt = wave % MT;                     // this wave's output channel block
    const int co0 = mt * 16 + g * 4;              // the lane's first output channel

    // ---- A fragments of both convolutions for rows mt*16 .. +15: A[o][k] = w[tap][i][o]
    // with k = tap*C + i (zero past the 9 taps); biases of the lane's four output channels
    // (the loads of one convolution all in flight, from clamped rows: a launch on few frames
    // spends most of its time up to here)
    uint4 wr1[KSTEPS], wr2[KSTEPS];
    auto load_w = [&](const float* w, uint4 (&wr)[KSTEPS]) CB_INLINE_LAMBDA {
        const int o = mt * 16 + r16;
        float v[KSTEPS][8];
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int k = ks * 32 + g * 8 + j;
                v[ks][j] = w[(k < G::K ? k : G::K - 1) * C + o];
            }
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
            wr[ks] = make_uint4(pack2bf(v[ks][0], v[ks][1]), pack2bf(v[ks][2], v[ks][3]), pack2bf(v[ks][4], v[ks][5]), pack2bf(v[ks][6], v[ks][7]));
            if (ks * 32 + 31 >= G::K && ks * 32 + g * 8 >= G::K) wr[ks] = make_uint4(0, 0, 0, 0);
        }
    };
    load_w(a.w1, wr1);
    load_w(a.w2, wr2);
    float b1[4], b2[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        b1[j] = a.b1 ? a.b1[co0 + j] : 0.f;
        b2[j] = a.b2 ? a.b2[co0 + j] : 0.f;
    }
    // Per-lane B-fragment offsets from the tap-(0,0) pixel: a k-step spans two taps, lane group g
    // the half (g & 1) of tap 2 ks + g / 2's 32 bytes; groups g >= 2 of the last k-step are past the
    // 9 taps and read the zero word.
    int boff[KSTEPS];
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
        const int tap = ks * 2 + (g >> 1);
        boff[ks] = ((tap / 3) * TW + tap % 3) * PXB + (g & 1) * 16;
    }
    const bool zsel = g >= 2;
    auto mma = [&](const unsigned char* xb, const unsigned char* zp, const uint4* wr) {
        cb_f32x4 acc = cb_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
            const unsigned char* p = ks == KSTEPS - 1 && zsel ? zp : xb + boff[ks];
            acc = PrecBF16::mma(wr[ks], *reinterpret_cast<const uint4*>(p), acc);
        }
        return acc;
    };

    // ---- relu(t) window and zero word cleared once (padding columns are never written)
    for (int j = tid; j < G::twin_bytes(TH, W) / 16; j += NT) reinterpret_cast<uint4*>(tw)[j] = make_uint4(0, 0, 0, 0);

    // ---- x-window staging offsets, tile-invariant per lane (slot k of this wave:
    // j = (wave + NW*k)*64 + lane, 16 bytes: plane, pixel, half), relative to image row 0; a
    // tile adds h0 - 2 rows. Rows off the frame fall outside the frame's buffer resource
    // (negative, or past its end); padding columns read zero (kOOB).
    const int npx = (TH + 4) * TW, nsx = MT * npx * 2;
    uint32_t ox[G::MAXS];
#pragma unroll
    for (int k = 0; k < G::MAXS; ++k) {
        const int j = (wave + NW * k) * 64 + lane, p = j >> 1, half = j & 1;
        const int rr = qdiv(p, t.inv_TW), col = p - rr * TW;
        const uint32_t off = uint32_t(((rr * W + col - 1) * C + half * 8) * 2);
        ox[k] = (j < nsx) & (uint32_t(col - 1) < uint32_t(W)) ? off : kOOB;
    }
    __syncthreads();

    int lg = blockIdx.x;   // neighbouring bands on one XCD
    if ((gridDim.x & 7) == 0) lg = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);

    // x window of a tile, rows h0-2 .. h0+TH+1. The next tile's window is issued as soon as
    // conv1 has finished reading this one, so its latency overlaps conv2.
    auto stage_x = [&](unsigned char* dst, int tile) {
        const int band = tile % t.nbands, f = tile / t.nbands;
        const auto rx = buf_rsrc(static_cast<const uint16_t*>(a.x) + int64_t(f) * H * W * C, uint32_t(H) * W * C * 2);
        const uint32_t hr = uint32_t((band * TH - 2) * W * C * 2);   // wraps for h0 < 2: rows off the frame
#pragma unroll
        for (int k = 0; k < G::MAXS; ++k)
            if ((wave + NW * k) * 64 < nsx) dma16_to_lds(rx, dst + (wave + NW * k) * 1024, ox[k] + hr);
    };
    if (lg < t.ntiles) stage_x(xw, lg);

    for (int tile = lg; tile < t.ntiles; tile += gridDim.x) {
        const int band = tile % t.nbands, f = tile / t.nbands;
        const int h0 = band * TH, the = H - h0 < TH ? H - h0 : TH;
        const int64_t fo = int64_t(f) * H * W * C;   // frame offset (elements)
        // conv2's outputs: window pixels 1 .. (the-1)*TW + W of the band's rows (row-major,
        // padding columns included and dropped); pixel pw is band row pw / TW, column pw % TW - 1
        const uint16_t* xbase = static_cast<const uint16_t*>(a.x) + fo + int64_t(h0) * W * C;
        const int npx2 = the * TW - 2;
        auto y_px = [&](int q, int& rb, int& cw) {   // clamped window pixel of conv2 output q
            const int pw = 1 + (q < npx2 ? q : npx2 - 1);
            rb = qdiv(pw, t.inv_TW);
            cw = pw - rb * TW;
            return pw;
        };
        auto res_off = [&](int rb, int cw) {   // residual x of that pixel (columns clamped)
            const int c = cw < 1 ? 1 : (cw > W ? W : cw);
            return uint32_t((rb * W + c - 1) * C + co0);
        };
        __builtin_amdgcn_s_waitcnt(0);   // this tile's window has landed
        __syncthreads();
        // conv2's residual for this wave's column tiles, in flight during the ReLU pass and conv1
        uint2 xres[G::MAXT];
#pragma unroll
        for (int k = 0; k < G::MAXT; ++k) {
            const int q = (wave / MT + k * (NW / MT)) * 16 + r16;
            int rb, cw;
            y_px(q, rb, cw);
            xres[k] = *reinterpret_cast<const uint2*>(xbase + res_off(rb, cw));
        }
        {
            uint4* w4 = reinterpret_cast<uint4*>(xw);
            for (int j = tid; j < nsx; j += NT) {
                uint4 v = w4[j];
                v.x = relu_bf16x2(v.x); v.y = relu_bf16x2(v.y); v.z = relu_bf16x2(v.z); v.w = relu_bf16x2(v.w);
                w4[j] = v;
            }
        }
        // t rows tr of the window <-> image row h0 - 1 + tr; rows outside the image stay zero
        const int tr0 = h0 == 0 ? 1 : 0;
        const int tr1 = the + 2 < H - h0 + 1 ? the + 2 : H - h0 + 1;
        {
            const int row16 = TW * PXB / 16;
            for (int pl = 0; pl < MT; ++pl) {
                uint4* t4 = reinterpret_cast<uint4*>(tw + pl * tps);
                if (tr0 == 1)
                    for (int j = tid; j < row16; j += NT) t4[j] = make_uint4(0, 0, 0, 0);
                for (int j = tid; j < (the + 2 - tr1) * row16; j += NT) t4[tr1 * row16 + j] = make_uint4(0, 0, 0, 0);
            }
        }
        __syncthreads();

        // ---- conv1: t on window rows [tr0, tr1), window pixels tr0*TW + 1 .. (tr1-1)*TW + W
        uint16_t* tbase = static_cast<uint16_t*>(a.t) + fo;
        const int npx1 = (tr1 - tr0) * TW - 2, pw1 = tr0 * TW + 1;
        for (int nt = wave / MT; nt * 16 < npx1; nt += NW / MT) {
            const int q = nt * 16 + r16;
            const int pw = pw1 + (q < npx1 ? q : npx1 - 1);
            const int tr = qdiv(pw, t.inv_TW), cw = pw - tr * TW;
            const cb_f32x4 acc = mma(xw + (pw - 1) * PXB, tw + MT * tps, wr1);   // tap (0,0): x-window pixel pw - 1
            if (q < npx1 && cw >= 1 && cw <= W) {
                const int h = h0 - 1 + tr;
                const uint32_t u0 = pack2bf(acc[0] + b1[0], acc[1] + b1[1]);
                const uint32_t u1 = pack2bf(acc[2] + b1[2], acc[3] + b1[3]);
                if (h >= h0 && h < h0 + the)
                    *reinterpret_cast<uint2*>(tbase + (uint32_t(h) * W + cw - 1) * C + co0) = make_uint2(u0, u1);
                *reinterpret_cast<uint2*>(tw + mt * tps + pw * PXB + g * 8) = make_uint2(relu_bf16x2(u0), relu_bf16x2(u1));
            }
        }
        __syncthreads();   // conv1 has read the x window: the next tile's may land there

        // ---- next tile's x window, then conv2 + residual (y on the band's rows). The two
        // windows are restrict parameters of one call, so the compiler knows that the loads in
        // flight into the x window do not write the relu(t) window that conv2 reads, and does
        // not wait for them before conv2's LDS reads.
        auto stage_conv2 = [&](unsigned char* __restrict__ xdst, const unsigned char* __restrict__ tsrc) {
            if (tile + int(gridDim.x) < t.ntiles) stage_x(xdst, tile + gridDim.x);
            uint16_t* ybase = static_cast<uint16_t*>(a.y) + fo + int64_t(h0) * W * C;
            auto conv2_tile = [&](int nt, const uint2& xr) {
                const int q = nt * 16 + r16;
                int rb, cw;
                const int pw = y_px(q, rb, cw);
                const cb_f32x4 acc = mma(tsrc + (pw - 1) * PXB, tsrc + MT * tps, wr2);   // tap (0,0): t-window pixel pw - 1
                if (q < npx2 && cw >= 1 && cw <= W)
                    store4(ybase + uint32_t((rb * W + cw - 1) * C + co0), acc[0] + b2[0] + __uint_as_float(xr.x << 16),
                           acc[1] + b2[1] + __uint_as_float(xr.x & 0xffff0000u),
                           acc[2] + b2[2] + __uint_as_float(xr.y << 16),
                           acc[3] + b2[3] + __uint_as_float(xr.y & 0xffff0000u));
            };
#pragma unroll
            for (int k = 0; k < G::MAXT; ++k)
                if ((wave / MT + k * (NW / MT)) * 16 < npx2) conv2_tile(wave / MT + k * (NW / MT), xres[k]);
        };
        stage_conv2(xw, tw);
    }
}

// The 32-channel block by column walks. What bounded the tile-by-tile form was LDS: a 3x3
// convolution with one B fragment (16 pixels x 32 channels, 1 KB) read per tap and output block
// reads 1 KB of LDS per MFMA, more than the LDS delivers at the matrix cores' rate. Here the 16
// pixels of a fragment are 16 anchors (a column of the band, or a segment of it), and a wave
// walks its anchors down the rows: the three fragments of an input row (kx = 0, 1, 2) feed the
// three output rows they touch, both 16-channel output blocks each, 18 MFMAs for 3 KB, and the
// next row's three are read meanwhile. Each wave holds both convolutions' weights for both
// output blocks (144 registers): two 4-wave workgroups per CU, each with its own windows (one, with windows
// of twice the size, where a frame is too wide: MAXS slots per lane).
// Sums keep the tap order of one output pixel's chain, so results are those of the per-layer
// convolutions bit for bit.
//   - One padding column serves both sides (the right neighbour of a row's last pixel is the next
//     row's padding); walk.h has the windows' layout.
//   - The x window stays as loaded (the fragments are ReLU'd in registers), so the residual comes
//     from LDS too, and nothing is read twice from memory but a band's halo rows.
//   - Output rows of the A operand are permuted so that lane group g receives channels 8g .. 8g+7:
//     one 16-byte store per pixel, 1 KB contiguous per wave.
//   - The weights are read once per workgroup, coalesced, and shared through LDS.
// Measured against a tile-by-tile form (at 42x42 against a two-role pipelined form of it), graph
// replays on one card: 2048 frames of 21x21 74 -> 43.6 us (2.3 -> 4.0 TB/s of its three tensors), 8192 260
// -> 155, 640 28.9 -> 21.3, 128 12.7 -> 8.5, 8 11.7 -> 5.3; 8192 of 42x42 969 -> 765, 2048 of 11x11 25.8 ->
// 17.9. With walks of one row, which reuse nothing, 21x21 takes 53 us. What is left at 21x21: about 2.6 us
// before the first row; then a tile's work and its loads, which add up unless the other workgroup covers
// them. (Tile shapes: walkplan.h.)
template <int R, int MAXS>
__global__ __launch_bounds__(RwGeom::NT, 2) void resblock_walk_fwd_kernel(ResBlockArgs a, RwTile t) {
    using G = RwGeom;
    constexpr int NT = G::NT, NW = G::NW, KS = G::KS, C = G::C;
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* xw = smem;                                  // x [F][TH+2+2ho][TW], row 0 = image row h0-1-ho
    unsigned char* tw = smem + t.t_off;                        // relu(t) [F][TH+2][TW], row 0 = image row h0-1

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, r16 = lane & 15;
    const int H = a.H, W = a.W, F = t.F, TH = t.TH, ho = t.ho, TW = walk_pitch(W);
    const int xrows = TH + 2 + 2 * ho, trows = TH + 2, xpf = xrows * TW, tpf = trows * TW;
    const int nsx = (F * xpf + 1) * 4;                         // x-window 16-byte slots staged
    const int rowb = TW * 64;

    // ---- weights: 4 k-values x 4 output channels per unit, in flight while the offsets are formed
    // and packed below into A fragments in LDS (the t window's memory): fragment (conv, b, ks)
    // holds at lane 16 (k % 32 / 8) + i, i = 4 (o / 8) + o % 4, b = o / 4 % 2, the k-values
    // 8 (lane / 16) .. +7 of output channel o
    constexpr int UNITS = 2 * 9 * C / 4 * (C / 4), PER = (UNITS + NT - 1) / NT;
    float4 v[PER][4];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int id0 = tid + u * NT, id = id0 < UNITS ? id0 : UNITS - 1;   // clamped: loads without a branch
        const int cv = id >= UNITS / 2, r = id - cv * (UNITS / 2), k4 = r / (C / 4), o4 = r % (C / 4);
        const float* src = (cv ? a.w2 : a.w1) + k4 * 4 * C + o4 * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[u][i] = load_f4(src + i * C);
    }
    // biases of the lane's channels 8g .. 8g+7 (loaded from a valid address where there are none)
    float4 bias1[2], bias2[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        bias1[k] = load_f4((a.b1 ? a.b1 : a.w1) + g * 8 + 4 * k);
        bias2[k] = load_f4((a.b2 ? a.b2 : a.w1) + g * 8 + 4 * k);
    }
    // ---- x-window staging offsets, tile-invariant per lane (slot k of this wave: j = (wave +
    // NW*k)*64 + lane: pixel j / 4, position j % 4), relative to the tile's first frame with the
    // window's first row at image row 0; a tile adds that row. Rows off the frame fall outside
    // the tile's buffer resource (F > 1: they are kOOB); padding columns are kOOB and read zero.
    uint32_t ox[MAXS];
#pragma unroll
    for (int k = 0; k < MAXS; ++k) {
        const int j = (wave + NW * k) * 64 + lane, p = j >> 2;
        const int fi = qdiv(p, t.inv_xpf), pr = p - fi * xpf, rr = qdiv(pr, t.inv_TW), col = pr - rr * TW;
        const int q = (j & 3) ^ ((col >> 1) & 2);
        const int h = rr - (ho ? 0 : 1);   // whole frames: the window's first row is off the frame
        const bool in = (j < nsx) & (uint32_t(col - 1) < uint32_t(W)) & ((ho != 0) | (uint32_t(h) < uint32_t(H)));
        const uint32_t off = uint32_t((((fi * H + h) * W + col - 1) * C + q * 8) * 2);
        ox[k] = in ? off : kOOB;
    }
    int lg = blockIdx.x;   // neighbouring bands on one XCD
    if ((gridDim.x & 7) == 0) lg = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    auto stage_x = [&](int tile) {
        const int band = tile % t.nbands, f = (tile / t.nbands) * F;
        const int nf = a.n - f < F ? a.n - f : F;
        const auto rx = buf_rsrc(static_cast<const uint16_t*>(a.x) + int64_t(f) * H * W * C, uint32_t(nf) * H * W * C * 2);
        const uint32_t hr = ho ? uint32_t((band * TH - 2) * W * C * 2) : 0u;   // wraps for h0 < 2: rows off the frame
#pragma unroll
        for (int k = 0; k < MAXS; ++k)
            if ((wave + NW * k) * 64 < nsx) dma16_to_lds(rx, xw + (wave + NW * k) * 1024, ox[k] + hr);
    };
    if (lg < t.ntiles) stage_x(lg);

    uint4 w1[2][KS], w2[2][KS];
    {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int id = tid + u * NT, cv = id >= UNITS / 2, r = id - cv * (UNITS / 2), k4 = r / (C / 4), o4 = r % (C / 4);
            if (id < UNITS) {
                const int ks = k4 / 8, gk = (k4 % 8) / 2, hf = k4 & 1, b = o4 & 1, i0 = 4 * (o4 >> 1);
                unsigned char* dst = tw + cv * G::WFRAG + ((b * KS + ks) * 64 + gk * 16 + i0) * 16 + hf * 8;
                const float* f = reinterpret_cast<const float*>(v[u]);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    *reinterpret_cast<uint2*>(dst + j * 16) = make_uint2(pack2bf(f[j], f[4 + j]), pack2bf(f[8 + j], f[12 + j]));
            }
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (!a.b1) bias1[k] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (!a.b2) bias2[k] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        lds_barrier();
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                w1[b][ks] = *reinterpret_cast<const uint4*>(tw + ((b * KS + ks) * 64 + lane) * 16);
                w2[b][ks] = *reinterpret_cast<const uint4*>(tw + G::WFRAG + ((b * KS + ks) * 64 + lane) * 16);
            }
        lds_barrier();
        // the relu(t) window: its padding column and, for whole frames, its rows off the frame
        // are never written
        for (int j = tid; j < walk_win_bytes(64, F, trows, W) / 16; j += NT) reinterpret_cast<uint4*>(tw)[j] = make_uint4(0, 0, 0, 0);
    }

    const int cols = F * W;
    auto anchor = [&](int grp, int nseg, int nrows) {
        return walk_anchor(grp * 16 + r16, cols, W, nseg, R, nrows, t.inv_c, t.inv_W);
    };

    for (int tile = lg; tile < t.ntiles; tile += gridDim.x) {
        const int band = tile % t.nbands, f = (tile / t.nbands) * F;
        const int h0 = band * TH, the = H - h0 < TH ? H - h0 : TH;
        const int nf = a.n - f < F ? a.n - f : F;
        const int64_t fo = int64_t(f) * H * W * C;
        __builtin_amdgcn_s_waitcnt(0);   // this tile's window has landed
        __syncthreads();

        // ---- conv1: t on rows h0-ho .. h0+TH+ho-1 of every column
        {
            const int n1 = TH + 2 * ho;
            uint16_t* tbase = static_cast<uint16_t*>(a.t) + fo;
            for (int grp = wave; grp * 16 < t.nseg1 * cols; grp += NW) {
                const WalkAnchor an = anchor(grp, t.nseg1, n1);
                uint32_t ta = uint32_t(an.fi * tpf + (an.row0 + 1 - ho) * TW + an.c + 1) * 64 + walk_ch(an.c + 1, g * 16);
                const int hb = h0 - ho + an.row0;   // image row of the walk's first row
                uint32_t go = uint32_t(((an.fi * H + hb) * W + an.c) * C + g * 8);   // wraps above the frame, not stored
                const bool own = an.ok && an.fi < nf;
                walk_conv32<R, true>(xw, an.fi * xpf + an.row0 * TW + an.c, an.c, g, rowb, w1, [] {},
                    [&](int j, const cb_f32x4 (&acc)[2]) {
                        const float4 ba = bias1[0], bb = bias1[1];
                        uint4 u = make_uint4(pack2bf(acc[0][0] + ba.x, acc[0][1] + ba.y), pack2bf(acc[0][2] + ba.z, acc[0][3] + ba.w),
                                             pack2bf(acc[1][0] + bb.x, acc[1][1] + bb.y), pack2bf(acc[1][2] + bb.z, acc[1][3] + bb.w));
                        const int h = hb + j;
                        const bool mine = an.row0 + j >= an.rbeg;
                        if (own && mine && h >= h0 && h < h0 + the) store16(tbase + go, u);
                        u.x = relu_bf16x2(u.x); u.y = relu_bf16x2(u.y); u.z = relu_bf16x2(u.z); u.w = relu_bf16x2(u.w);
                        if (ho && (h < 0 || h >= H)) u = make_uint4(0, 0, 0, 0);   // conv2's zero padding
                        if (an.ok && mine) *reinterpret_cast<uint4*>(tw + ta) = u;
                        ta += rowb;
                        go += W * C;
                    });
            }
        }
        __syncthreads();   // the relu(t) window is complete

        // ---- conv2 + bias + residual: y on the band's rows
        {
            uint16_t* ybase = static_cast<uint16_t*>(a.y) + fo;
            for (int grp = wave; grp * 16 < t.nseg2 * cols; grp += NW) {
                const WalkAnchor an = anchor(grp, t.nseg2, TH);
                uint32_t xa = uint32_t(an.fi * xpf + (an.row0 + 1 + ho) * TW + an.c + 1) * 64 + walk_ch(an.c + 1, g * 16);
                uint32_t go = uint32_t(((an.fi * H + h0 + an.row0) * W + an.c) * C + g * 8);
                const bool own = an.ok && an.fi < nf;
                uint4 xr = make_uint4(0, 0, 0, 0);
                walk_conv32<R, false>(tw, an.fi * tpf + an.row0 * TW + an.c, an.c, g, rowb, w2,
                    [&] {
                        xr = *reinterpret_cast<const uint4*>(xw + xa);
                        xa += rowb;
                    },
                    [&](int j, const cb_f32x4 (&acc)[2]) {
                        const float4 ba = bias2[0], bb = bias2[1];
                        if (own && an.row0 + j >= an.rbeg && an.row0 + j < the)
                            store16(ybase + go,
                                make_uint4(pack2bf(acc[0][0] + ba.x + bf_lo(xr.x), acc[0][1] + ba.y + bf_hi(xr.x)),
                                           pack2bf(acc[0][2] + ba.z + bf_lo(xr.y), acc[0][3] + ba.w + bf_hi(xr.y)),
                                           pack2bf(acc[1][0] + bb.x + bf_lo(xr.z), acc[1][1] + bb.y + bf_hi(xr.z)),
                                           pack2bf(acc[1][2] + bb.z + bf_lo(xr.w), acc[1][3] + bb.w + bf_hi(xr.w))));
                        go += W * C;
                    });
            }
        }
        __syncthreads();   // both windows have been read
        if (tile + int(gridDim.x) < t.ntiles) stage_x(tile + gridDim.x);
    }
}

namespace {

constexpr size_t kRbLds = 160 * 1024;   // per CU, shared by the resident workgroups

template <int C>
hipError_t rb_fwd_launch(const ResBlockArgs& a, hipStream_t s) {
    using G = RbGeom<C>;
    constexpr int kRbWaves = G::NW;
    constexpr size_t kRbLdsTarget = kRbLds / G::WGS;
    const int H = a.H, W = a.W;
    auto lds = [&](int th) { return size_t(G::xwin_bytes(th, W)) + G::twin_bytes(th, W); };
    auto fits = [&](int th) {
        const int tiles = (th * (W + 2) - 2 + 15) / 16, per = kRbWaves / G::MT;
        return G::blocks(G::MT * (th + 4) * (W + 2) * 2) <= G::MAXS * kRbWaves && (tiles + per - 1) / per <= G::MAXT;
    };
    int thmax = H;
    while (thmax > 1 && (lds(thmax) > kRbLdsTarget || !fits(thmax))) --thmax;
    if (lds(thmax) > std::min<size_t>(lds_limit(), 160 * 1024) || !fits(thmax)) return hipErrorInvalidValue;
    if (int64_t(H) * W * C * 2 >= (int64_t(1) << 31)) return hipErrorInvalidValue;
    int TH = 1, best = 1 << 30;   // fewest staged window rows per frame
    for (int th = 1; th <= thmax; ++th) {
        const int rows = (H + th - 1) / th * (th + 4);
        if (rows <= best) { best = rows; TH = th; }
    }
    RbTile t{};
    t.TH = TH; t.nbands = (H + TH - 1) / TH; t.ntiles = t.nbands * a.n;
    t.x_off = 0;
    t.t_off = G::xwin_bytes(TH, W);
    t.inv_W = 1.f / float(W); t.inv_TW = 1.f / float(W + 2);
    const size_t L = lds(TH);
    const void* fn = reinterpret_cast<const void*>(&resblock_fwd_kernel<C, kRbWaves>);
    int gx = std::max(1, resident_blocks(fn, 64 * kRbWaves, L));
    if (gx > t.ntiles) gx = t.ntiles;
    ProfScope ps(s, [&] { return cb_key("resblock_fwd", 0, cb_dims(C, C) + "/" + cb_dims(H, W)); });
    hipLaunchKernelGGL((resblock_fwd_kernel<C, kRbWaves>), dim3(unsigned(gx)), dim3(64 * kRbWaves), L, s, a, t);
    return hipGetLastError();
}

hipError_t rw_launch(const ResBlockArgs& a, hipStream_t s) {
    using G = RwGeom;
    const int H = a.H, W = a.W, cus = device_cus();
    if (int64_t(H) * W * G::C * 2 >= (int64_t(1) << 31)) return hipErrorInvalidValue;
    static thread_local WalkPlans<RwTile> plans;
    const auto* plan = plans.find(a.n, H, W, cus);
    if (!plan) {
        RwTile t{};
        size_t L = 0;
        if (!walk_choose([&](auto&& f) { rw_shapes(a.n, H, W, cus, f); }, t, L)) return hipErrorInvalidValue;
        plan = plans.put({a.n, H, W, cus, t, L});
    }
    auto launch = [&](auto r, auto slots) {
        constexpr int R = decltype(r)::value, MAXS = decltype(slots)::value;
        const void* fn = reinterpret_cast<const void*>(&resblock_walk_fwd_kernel<R, MAXS>);
        const int gx = std::min(plan->t.ntiles, std::max(1, resident_blocks(fn, G::NT, plan->lds)));
        ProfScope ps(s, [&] { return cb_key("resblock_fwd", 0, cb_dims(G::C, G::C) + "/" + cb_dims(H, W)); });
        hipLaunchKernelGGL((resblock_walk_fwd_kernel<R, MAXS>), dim3(unsigned(gx)), dim3(G::NT), plan->lds, s, a, plan->t);
    };
    if (plan->t.wide) walk_dispatch<G::WIDE_MAXR>(plan->t.R, [&](auto r) { launch(r, std::integral_constant<int, G::WIDE_MAXS>{}); });
    else walk_dispatch<G::MAXR>(plan->t.R, [&](auto r) { launch(r, std::integral_constant<int, G::MAXS>{}); });
    return hipGetLastError();
}

}  // namespace

bool resblock_fwd_supported(int C) { return C == 16 || C == 32; }

hipError_t resblock_fwd(int C, const ResBlockArgs& a, hipStream_t s) {
    if (a.n <= 0) return hipSuccess;
    if (C == 16) return rb_fwd_launch<16>(a, s);
    if (C == 32) return rw_launch(a, s);
    return hipErrorInvalidValue;
}

}  // namespace cb
