// Backward pass of a whole IMPALA-ResNet residual block (Section 5's network) in one kernel,
// bf16 storage and float32 accumulation on gfx950 MFMA. With the block's forward
//
//   t = conv_a(relu(x)) + b_a,   y = x + conv_b(relu(t)) + b_b     (3x3 SAME convolutions, C -> C)
//
// and the gradient dy at its output:
//
//   dt  = conv_b^T(dy) * [t > 0]           dWb = sum_p relu(t)[p + d(tap)] dy[p],  dbb = sum_p dy[p]
//   dx  = conv_a^T(dt) * [x > 0] + dy      dWa = sum_p relu(x)[p + d(tap)] dt[p],  dba = sum_p dt[p]
//
// As two fused conv backward launches this moves seven activation tensors through HBM (dy and
// t in, dt out; dt, x and dy in, dx out). Here dt is formed in an LDS window, rounded to bf16 as the
// two-launch path stores it (a band of a frame forms one halo row either side, which the
// neighbouring bands form too), and four tensors move: dy, t and x in, dx out.
//
// The input-gradient weights (taps rotated by 180 degrees, channels swapped) live in registers; the
// weight gradients accumulate in registers over all tiles of a workgroup; each workgroup writes one
// float32 partial per conv, summed in a fixed order by a later launch (deterministic, no atomics).
#include "common.h"
#include "kernels.h"
#include "walk.h"

#include <algorithm>
#include <type_traits>

namespace cb {

// The 32-channel block backward by column walks (walk.h), in one 8-wave workgroup per CU with
// two wave roles. Waves 0-3 form dt, then dx, for both channel blocks (both convolutions' weights:
// 144 registers; each input fragment feeds 18 MFMAs); waves 4-7 form conv_b's weight gradient
// while dt is formed and conv_a's beside dx, each wave one 16x16 channel block of all nine taps (18
// tap tiles and the bias columns: 80 registers; each x fragment feeds three rows of dy). A tile (F
// whole frames, or a band of one) has two phases:
//   a: dt = conv_b^T(dy) * [t > 0] into the dt window; dWb from dy and t; x and dy's own pixels
//      once more (for the skip term; an L2 hit) are being staged;
//   b: dx = conv_a^T(dt) * [x > 0] + dy; dWa from dt and x; the next tile's dy and t are staged.
// No phase reads what is being staged in it, so loads overlap all of the work with one set of
// windows in LDS.
// Measured against a form that read every fragment once per tap and block (its own two roles
// bound by LDS and by the vector instructions beside the MFMAs): 2048 frames of 21x21 138 -> 101 us,
// of 11x11 56 -> 45 us, 8192 of 42x42 1590 -> 1490 us, 640 of 11x11 with its reduce 36 -> 25 us.
// What bounds it: a SIMD's MFMAs (about 270 of 16 cycles per phase at 21x21) and the vector
// instructions of its two waves, which overlap 1.6 to 1; then staging and barriers.
// One window of a tile, HBM -> LDS: block wave + NW*k of 64 16-byte slots from the lane's offset
// off[k], shifted by `row` rows.
template <int C, int N>
CB_DEV void rbw_stage(const ResBwdArgs& a, const RbwTile& t, const void* src, unsigned char* win, int ns,
                      const uint32_t (&off)[N], int wave, int tile, int row) {
    constexpr int NW = RbwGeom::NW;
    const int band = tile % t.nbands, f = (tile / t.nbands) * t.F;
    const int nf = a.n - f < t.F ? a.n - f : t.F, fel = a.H * a.W * C;
    const auto r = buf_rsrc(static_cast<const uint16_t*>(src) + int64_t(f) * fel, uint32_t(nf) * fel * 2);
    const uint32_t hr = uint32_t((band * t.TH - row) * a.W * C * 2);   // wraps above the frame
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const int blk = wave + NW * k;
        if (blk * 64 < ns) dma16_to_lds(r, win + blk * 1024, off[k] + hr);
    }
}

// Waits for this wave's loads, then relu of the blocks it staged of a window, in place: before
// the barrier that shows them to the other waves, so it takes no barrier of its own. Both convs
// read relu'd inputs, and relu(v) > 0 exactly where v > 0, so the masks read them too.
template <int N>
CB_DEV void rbw_landed(unsigned char* win, int ns, int wave, int lane) {
    __builtin_amdgcn_s_waitcnt(0);
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const int blk = wave + RbwGeom::NW * k;
        if (blk * 64 < ns) {
            uint4* p = reinterpret_cast<uint4*>(win + blk * 1024) + lane;
            *p = relu8(*p);
        }
    }
}

template <int R>
__global__ __launch_bounds__(RbwGeom::NT, 2) void resblock_bwd_walk_kernel(ResBwdArgs a, RbwTile t) {
    using G = RbwGeom;
    constexpr int NT = G::NT, NW = G::NW, NS = G::NS, C = G::C;
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* dyw = smem;               // dy [F][TH+2+2ho][TW], row 0 = image row h0-1-ho
    unsigned char* tw = smem + t.t_off;      // relu(t) [F][TH+2][TW], row 0 = image row h0-1
    unsigned char* xw = smem + t.x_off;      // relu(x), likewise
    unsigned char* dtw = smem + t.dt_off;    // dt, likewise
    unsigned char* skw = smem + t.sk_off;    // dy's own pixels [F][TH][W]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool dgrad = wave < NS;            // input-gradient role
    const int rw = wave & (NS - 1);          // wave within its role
    const int H = a.H, W = a.W, F = t.F, TH = t.TH, ho = t.ho, TW = walk_pitch(W);
    const int dpf = (TH + 2 + 2 * ho) * TW, xpf = (TH + 2) * TW;
    const int nsd = (F * dpf + 1) * 4, nsx = (F * xpf + 1) * 4, nsk = F * TH * W * 4;   // 16-byte slots staged
    const int rowb = TW * 64, cols = F * W;

    // ---- staging offsets, tile-invariant per lane (slot k of this wave: j = (wave + NW*k)*64 +
    // lane: pixel j / 4, position j % 4), relative to the tile's first frame with the window's
    // first row at image row 0 (whole frames: at row -1); a tile adds that row. Rows off the frame fall
    // outside the buffer resource (whole frames: they are kOOB), padding columns are kOOB.
    uint32_t od[G::MAXD], ox[G::MAXX], ok[G::MAXK];
    auto win_off = [&](int j, int ns, int pf, float inv_pf) CB_INLINE_LAMBDA {
        const int p = j >> 2, fi = qdiv(p, inv_pf), pr = p - fi * pf, rr = qdiv(pr, t.inv_TW), col = pr - rr * TW;
        const int q = (j & 3) ^ ((col >> 1) & 2);
        const int h = rr - (ho ? 0 : 1);
        const bool in = (j < ns) & (uint32_t(col - 1) < uint32_t(W)) & ((ho != 0) | (uint32_t(h) < uint32_t(H)));
        const uint32_t off = uint32_t((((fi * H + h) * W + col - 1) * C + q * 8) * 2);
        return in ? off : kOOB;
    };
    const int rd = ho ? 2 : 0, rx = ho ? 1 : 0;   // a window's first row above the band (whole frames: in the offsets)

    int lg = blockIdx.x;   // neighbouring bands (which share halo rows) on one XCD
    if ((gridDim.x & 7) == 0) lg = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const int G0 = int(gridDim.x);

    // ---- weights, loaded first and packed below: 4 k-values (output channels of the forward) of one
    // input channel o per unit; A[o][tap * 32 + co] = w[8 - tap][o][co]
    constexpr int UNITS = 2 * 9 * C * (C / 4), PER = UNITS / NT;
    static_assert(UNITS % NT == 0, "whole units per thread");
    float4 v[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int id = tid + u * NT, cv = id >= UNITS / 2, r = id - cv * (UNITS / 2);   // r = ((tap * 32) + o) * 8 + co / 4
        v[u] = load_f4((cv ? a.wb : a.wa) + r * 4);
    }
#pragma unroll
    for (int k = 0; k < G::MAXD; ++k) od[k] = win_off((wave + NW * k) * 64 + lane, nsd, dpf, t.inv_dpf);
#pragma unroll
    for (int k = 0; k < G::MAXX; ++k) ox[k] = win_off((wave + NW * k) * 64 + lane, nsx, xpf, t.inv_xpf);
#pragma unroll
    for (int k = 0; k < G::MAXK; ++k) {   // slot j: pixel j / 4 of the own pixels, permuted by its column
        const int j = (wave + NW * k) * 64 + lane, p = j >> 2;
        const int col = p - qdiv(p, t.inv_W) * W + 1, q = (j & 3) ^ ((col >> 1) & 2);
        ok[k] = j < nsk ? uint32_t(p * 64 + q * 16) : kOOB;
    }
    rbw_stage<C>(a, t, a.dy, dyw, nsd, od, wave, lg, rd);
    rbw_stage<C>(a, t, a.t, tw, nsx, ox, wave, lg, rx);
    // earlier launches' weight-gradient partials
    if (a.pend.nparts > 0) pending_reduce<NT>(a.pend, dtw);
    if (a.pend2.nparts > 0) pending_reduce<NT>(a.pend2, dtw);
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int id = tid + u * NT, cv = id >= UNITS / 2, r = id - cv * (UNITS / 2);
        const int ks = 8 - r / (C * 8), o = r / 8 % C, c4 = r % 8;   // k-step (rotated tap), row, 4-channel group
        *reinterpret_cast<uint2*>(dtw + cv * G::WFRAG + ((((o >> 2) & 1) * 9 + ks) * 64 + (c4 >> 1) * 16 + 4 * (o >> 3) + (o & 3)) * 16 +
                                  (c4 & 1) * 8) = make_uint2(pack2bf(v[u].x, v[u].y), pack2bf(v[u].z, v[u].w));
    }
    lds_barrier();
    // the dt window: its padding and, for whole frames, its rows off the frame are never written
    auto clear_dt = [&] {
        for (int j = tid; j < t.dt_bytes / 16; j += NT) reinterpret_cast<uint4*>(dtw)[j] = make_uint4(0, 0, 0, 0);
    };

    if (dgrad) {
        uint4 wa[2][9], wb[2][9];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int ks = 0; ks < 9; ++ks) {
                wa[b][ks] = *reinterpret_cast<const uint4*>(dtw + ((b * 9 + ks) * 64 + lane) * 16);
                wb[b][ks] = *reinterpret_cast<const uint4*>(dtw + G::WFRAG + ((b * 9 + ks) * 64 + lane) * 16);
            }
        lds_barrier();
        clear_dt();
        for (int tile = lg; tile < t.ntiles; tile += G0) {
            int ln = lane;
            asm volatile("" : "+v"(ln));   // anchors and row masks are formed per tile: kept over tiles they spill
            const int g = ln >> 4, r16 = ln & 15;
            const int band = tile % t.nbands, f = (tile / t.nbands) * F;
            const int h0 = band * TH, the = H - h0 < TH ? H - h0 : TH;
            const int nf = a.n - f < F ? a.n - f : F;
            const int64_t fo = int64_t(f) * H * W * C;
            rbw_landed<G::MAXX>(tw, nsx, wave, lane);
            lds_barrier();   // dy and t have landed; x and dt of the previous tile have been read
            // (the windows being staged and those read are restrict parameters of one call, so the
            // compiler knows that the loads in flight do not write what is read)
            auto phase_a = [&](unsigned char* __restrict__ xdst, unsigned char* __restrict__ kdst, unsigned char* __restrict__ dtdst,
                               const unsigned char* __restrict__ dsrc, const unsigned char* __restrict__ tsrc) CB_INLINE_LAMBDA {
                rbw_stage<C>(a, t, a.x, xdst, nsx, ox, wave, tile, rx);
                rbw_stage<C>(a, t, a.dy, kdst, nsk, ok, wave, tile, 0);
                const int n1 = TH + 2 * ho;
                for (int grp = rw; grp * 16 < t.nsegt * cols; grp += NS) {
                    const WalkAnchor an = walk_anchor(grp * 16 + r16, cols, W, t.nsegt, R, n1, t.inv_c, t.inv_W);
                    uint32_t ta = uint32_t(an.fi * xpf + (an.row0 + 1 - ho) * TW + an.c + 1) * 64 + walk_ch(an.c + 1, g * 16);
                    const int hb = h0 - ho + an.row0;   // image row of the walk's first row
                    const uint32_t one = 0x00010001u, top = 0x7f807f80u;
                    uint4 mk = make_uint4(0, 0, 0, 0);
                    walk_conv32<R, false>(dsrc, an.fi * dpf + an.row0 * TW + an.c, an.c, g, rowb, wb,
                        [&] { mk = *reinterpret_cast<const uint4*>(tsrc + ta); },
                        [&](int j, const cb_f32x4 (&acc)[2]) {
                            const int h = hb + j;
                            const bool in = uint32_t(h) < uint32_t(H);   // rows off the frame stay zero
                            uint4 u = make_uint4(pos_mask16x2(mk.x, pack2bf(acc[0][0], acc[0][1]), one, top), pos_mask16x2(mk.y, pack2bf(acc[0][2], acc[0][3]), one, top),
                                                 pos_mask16x2(mk.z, pack2bf(acc[1][0], acc[1][1]), one, top), pos_mask16x2(mk.w, pack2bf(acc[1][2], acc[1][3]), one, top));
                            if (!in) u = make_uint4(0, 0, 0, 0);
                            if (an.ok && an.row0 + j >= an.rbeg) *reinterpret_cast<uint4*>(dtdst + ta) = u;
                            ta += rowb;
                        });
                }
            };
            phase_a(xw, skw, dtw, dyw, tw);
            rbw_landed<G::MAXX>(xw, nsx, wave, lane);
            lds_barrier();   // the dt window is complete, x has landed
            auto phase_b = [&](unsigned char* __restrict__ ddst, unsigned char* __restrict__ tdst, const unsigned char* __restrict__ dtsrc,
                               const unsigned char* __restrict__ xsrc, const unsigned char* __restrict__ ksrc) CB_INLINE_LAMBDA {
                if (tile + G0 < t.ntiles) {
                    rbw_stage<C>(a, t, a.dy, ddst, nsd, od, wave, tile + G0, rd);
                    rbw_stage<C>(a, t, a.t, tdst, nsx, ox, wave, tile + G0, rx);
                }
                uint16_t* dxb = static_cast<uint16_t*>(a.dx) + fo;
                for (int grp = rw; grp * 16 < t.nsegx * cols; grp += NS) {
                    const WalkAnchor an = walk_anchor(grp * 16 + r16, cols, W, t.nsegx, R, TH, t.inv_c, t.inv_W);
                    uint32_t xa = uint32_t(an.fi * xpf + (an.row0 + 1) * TW + an.c + 1) * 64 + walk_ch(an.c + 1, g * 16);
                    uint32_t ka = uint32_t((an.fi * TH + an.row0) * W + an.c) * 64 + walk_ch(an.c + 1, g * 16);
                    uint32_t go = uint32_t(((an.fi * H + h0 + an.row0) * W + an.c) * C + g * 8);
                    const bool own = an.ok && an.fi < nf;
                    uint4 mk = make_uint4(0, 0, 0, 0), sk = make_uint4(0, 0, 0, 0);
                    walk_conv32<R, false>(dtsrc, an.fi * xpf + an.row0 * TW + an.c, an.c, g, rowb, wa,
                        [&] {
                            mk = *reinterpret_cast<const uint4*>(xsrc + xa);
                            sk = *reinterpret_cast<const uint4*>(ksrc + ka);
                            xa += rowb;
                            ka += W * 64;
                        },
                        [&](int j, const cb_f32x4 (&acc)[2]) {
                            if (own && an.row0 + j >= an.rbeg && an.row0 + j < the)
                                store16(dxb + go,
                                    make_uint4(pack2bf((bf_lo(mk.x) > 0.f ? acc[0][0] : 0.f) + bf_lo(sk.x), (bf_hi(mk.x) > 0.f ? acc[0][1] : 0.f) + bf_hi(sk.x)),
                                               pack2bf((bf_lo(mk.y) > 0.f ? acc[0][2] : 0.f) + bf_lo(sk.y), (bf_hi(mk.y) > 0.f ? acc[0][3] : 0.f) + bf_hi(sk.y)),
                                               pack2bf((bf_lo(mk.z) > 0.f ? acc[1][0] : 0.f) + bf_lo(sk.z), (bf_hi(mk.z) > 0.f ? acc[1][1] : 0.f) + bf_hi(sk.z)),
                                               pack2bf((bf_lo(mk.w) > 0.f ? acc[1][2] : 0.f) + bf_lo(sk.w), (bf_hi(mk.w) > 0.f ? acc[1][3] : 0.f) + bf_hi(sk.w))));
                            go += W * C;
                        });
                }
            };
            phase_b(dyw, tw, dtw, xw, skw);
        }
        return;
    }

    // ---- weight-gradient role: channel blocks (co, ci) of this wave
    lds_barrier();
    clear_dt();
    const int cob = rw & 1, cib = rw >> 1;
    cb_f32x4 accA[9], accB[9], biasA, biasB;
#pragma unroll
    for (int k = 0; k < 9; ++k) accA[k] = accB[k] = cb_f32x4{0.f, 0.f, 0.f, 0.f};
    biasA = biasB = cb_f32x4{0.f, 0.f, 0.f, 0.f};
    // dwin's own row 0 is window row drow; xwin's row 0 is one image row above it
    auto wgrad = [&](const unsigned char* xwin, const unsigned char* dwin, int dstride, int drow, cb_f32x4 (&acc)[9], cb_f32x4& accb) CB_INLINE_LAMBDA {
        for (int grp = 0; grp * 64 < t.nsegw * cols; ++grp) {
            int ln = lane;
            asm volatile("" : "+v"(ln));   // (as above)
            const int g = ln >> 4, jj = (ln >> 2) & 3, m = ln & 3;
            const uint32_t cx = uint32_t(cib * 32 + m * 8), cd = uint32_t(cob * 32 + m * 8);
            int px[4], pd[4], c[4], skip[4];
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                const WalkAnchor an = walk_anchor(grp * 64 + h * 16 + 4 * g + jj, cols, W, t.nsegw, R, TH, t.inv_c, t.inv_W);
                px[h] = an.fi * xpf + an.row0 * TW + an.c;
                pd[h] = an.fi * dstride + (an.row0 + drow) * TW + an.c + 1;
                c[h] = an.c;
                skip[h] = an.ok ? an.rbeg - an.row0 : R;
            }
            walk_wgrad<R>(xwin, dwin, px, pd, c, skip, cx, cd, rowb, acc, accb);
        }
    };
    auto phase_a = [&](unsigned char* __restrict__ xdst, unsigned char* __restrict__ kdst, const unsigned char* __restrict__ tsrc,
                       const unsigned char* __restrict__ dsrc, int tile) CB_INLINE_LAMBDA {
        rbw_stage<C>(a, t, a.x, xdst, nsx, ox, wave, tile, rx);
        rbw_stage<C>(a, t, a.dy, kdst, nsk, ok, wave, tile, 0);
        wgrad(tsrc, dsrc, dpf, 1 + ho, accB, biasB);
    };
    auto phase_b = [&](unsigned char* __restrict__ ddst, unsigned char* __restrict__ tdst, const unsigned char* __restrict__ xsrc,
                       const unsigned char* __restrict__ dtsrc, int next) CB_INLINE_LAMBDA {
        if (next < t.ntiles) {
            rbw_stage<C>(a, t, a.dy, ddst, nsd, od, wave, next, rd);
            rbw_stage<C>(a, t, a.t, tdst, nsx, ox, wave, next, rx);
        }
        wgrad(xsrc, dtsrc, xpf, 1, accA, biasA);
    };
    for (int tile = lg; tile < t.ntiles; tile += G0) {
        rbw_landed<G::MAXX>(tw, nsx, wave, lane);
        lds_barrier();
        phase_a(xw, skw, tw, dyw, tile);
        rbw_landed<G::MAXX>(xw, nsx, wave, lane);
        lds_barrier();
        phase_b(dyw, tw, xw, dtw, tile + G0);
    }

    // ---- this workgroup's partials: conv_b's set, then conv_a's
    float* part = a.partial + int64_t(blockIdx.x) * G::PSTRIDE + cob * G::NBB * 256;
    const int g = lane >> 4, r16 = lane & 15;
    auto put = [&](float* dst, const cb_f32x4& acc) {
#pragma unroll
        for (int e = 0; e < 4; ++e) dst[(4 * g + e) * 16 + r16] = acc[e];
    };
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        put(part + (2 * k + cib) * 256, accB[k]);
        put(part + t.pset + (2 * k + cib) * 256, accA[k]);
    }
    if (cib == 0) put(part + 18 * 256, biasB);
    else put(part + t.pset + 18 * 256, biasA);
}

// The 16-channel block backward in the same form. One fragment of weight-gradient anchors fills a wave
// (all nine taps of the one channel block: 40 registers a convolution), so the four waves share the
// anchors and their sums are added at the end.
// Measured against a form of two workgroups per CU that staged a tile, waited, and read every
// fragment once per tap: 2048 frames of 42x42 152.5 -> 144.7 us, 640 of 42x42 60 -> 55.5 us, of 21x21
// 31.5 -> 26 us, of 11x11 22.7 -> 17.8 us. Two workgroups of this form per CU (80 KB windows, 128
// registers, which spill) were slower: 180 us on 2048 frames of 42x42. What bounds it: 462 MB at the
// rate of a large copy are 97 us; the rest is a phase's loads that outlast its work, and barriers.
template <int R>
__global__ __launch_bounds__(Rbw16Geom::NT, 2) void resblock_bwd16_walk_kernel(ResBwdArgs a, RbwTile t) {
    using G = Rbw16Geom;
    constexpr int NT = G::NT, NW = G::NW, NS = G::NS, C = G::C;
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* dyw = smem;               // dy [F][TH+2+2ho][TW], row 0 = image row h0-1-ho
    unsigned char* tw = smem + t.t_off;      // relu(t) [F][TH+2][TW], row 0 = image row h0-1
    unsigned char* xw = smem + t.x_off;      // relu(x), likewise
    unsigned char* dtw = smem + t.dt_off;    // dt, likewise
    unsigned char* skw = smem + t.sk_off;    // dy's own pixels [F][TH][W]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool dgrad = wave < NS;            // input-gradient role
    const int rw = wave & (NS - 1);          // wave within its role
    const int H = a.H, W = a.W, F = t.F, TH = t.TH, ho = t.ho, TW = walk_pitch(W);
    const int dpf = (TH + 2 + 2 * ho) * TW, xpf = (TH + 2) * TW;
    const int nsd = (F * dpf + 1) * 2, nsx = (F * xpf + 1) * 2, nsk = F * TH * W * 2;   // 16-byte slots staged
    const int rowb = TW * 32, cols = F * W;

    // ---- staging offsets, tile-invariant per lane (slot k of this wave: j = (wave + NW*k)*64 +
    // lane: pixel j / 2, half j % 2), relative to the tile's first frame with the window's
    // first row at image row 0 (whole frames: at row -1); a tile adds that row. Rows off the frame fall
    // outside the buffer resource (whole frames: they are kOOB), padding columns are kOOB.
    uint32_t od[G::MAXD], ox[G::MAXX], ok[G::MAXK];
    auto win_off = [&](int j, int ns, int pf, float inv_pf) CB_INLINE_LAMBDA {
        const int p = j >> 1, fi = qdiv(p, inv_pf), pr = p - fi * pf, rr = qdiv(pr, t.inv_TW), col = pr - rr * TW;
        const int h = rr - (ho ? 0 : 1);
        const bool in = (j < ns) & (uint32_t(col - 1) < uint32_t(W)) & ((ho != 0) | (uint32_t(h) < uint32_t(H)));
        const uint32_t off = uint32_t((((fi * H + h) * W + col - 1) * C + (j & 1) * 8) * 2);
        return in ? off : kOOB;
    };
    const int rd = ho ? 2 : 0, rx = ho ? 1 : 0;   // a window's first row above the band (whole frames: in the offsets)

    int lg = blockIdx.x;   // neighbouring bands (which share halo rows) on one XCD
    if ((gridDim.x & 7) == 0) lg = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const int G0 = int(gridDim.x);

#pragma unroll
    for (int k = 0; k < G::MAXD; ++k) od[k] = win_off((wave + NW * k) * 64 + lane, nsd, dpf, t.inv_dpf);
#pragma unroll
    for (int k = 0; k < G::MAXX; ++k) ox[k] = win_off((wave + NW * k) * 64 + lane, nsx, xpf, t.inv_xpf);
#pragma unroll
    for (int k = 0; k < G::MAXK; ++k) {   // the own pixels in memory order
        const int j = (wave + NW * k) * 64 + lane;
        ok[k] = j < nsk ? uint32_t(j * 16) : kOOB;
    }
    rbw_stage<C>(a, t, a.dy, dyw, nsd, od, wave, lg, rd);
    rbw_stage<C>(a, t, a.t, tw, nsx, ox, wave, lg, rx);
    // earlier launches' weight-gradient partials
    if (a.pend.nparts > 0) pending_reduce<NT>(a.pend, dtw);
    if (a.pend2.nparts > 0) pending_reduce<NT>(a.pend2, dtw);
    lds_barrier();
    // the dt window: its padding and, for whole frames, its rows off the frame are never written
    auto clear_dt = [&] {
        for (int j = tid; j < t.dt_bytes / 16; j += NT) reinterpret_cast<uint4*>(dtw)[j] = make_uint4(0, 0, 0, 0);
    };

    if (dgrad) {
        // A[o][tap * 16 + co] = w[8 - tap][o][co], zero past the 9 taps (loads clamped)
        uint4 wa[5], wb[5];
        auto load_w = [&](const float* w, uint4 (&wf)[5]) CB_INLINE_LAMBDA {
            const int g = lane >> 4, o = lane & 15;
            float4 v[5][2];
#pragma unroll
            for (int ks = 0; ks < 5; ++ks)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int tap = 2 * ks + (g >> 1);
                    v[ks][q] = load_f4(w + ((tap < 9 ? 8 - tap : 0) * C + o) * C + (g & 1) * 8 + 4 * q);
                }
#pragma unroll
            for (int ks = 0; ks < 5; ++ks) {
                wf[ks] = make_uint4(pack2bf(v[ks][0].x, v[ks][0].y), pack2bf(v[ks][0].z, v[ks][0].w), pack2bf(v[ks][1].x, v[ks][1].y),
                                    pack2bf(v[ks][1].z, v[ks][1].w));
                if (ks == 4 && g >= 2) wf[ks] = make_uint4(0, 0, 0, 0);
            }
        };
        load_w(a.wa, wa);
        load_w(a.wb, wb);
        lds_barrier();
        clear_dt();
        for (int tile = lg; tile < t.ntiles; tile += G0) {
            int ln = lane;
            asm volatile("" : "+v"(ln));   // anchors and row masks are formed per tile: kept over tiles they spill
            const int g = ln >> 4, r16 = ln & 15;
            const int band = tile % t.nbands, f = (tile / t.nbands) * F;
            const int h0 = band * TH, the = H - h0 < TH ? H - h0 : TH;
            const int nf = a.n - f < F ? a.n - f : F;
            const int64_t fo = int64_t(f) * H * W * C;
            rbw_landed<G::MAXX>(tw, nsx, wave, lane);
            lds_barrier();   // dy and t have landed; x and dt of the previous tile have been read
            // (the windows being staged and those read are restrict parameters of one call, so the
            // compiler knows that the loads in flight do not write what is read)
            auto phase_a = [&](unsigned char* __restrict__ xdst, unsigned char* __restrict__ kdst, unsigned char* __restrict__ dtdst,
                               const unsigned char* __restrict__ dsrc, const unsigned char* __restrict__ tsrc) CB_INLINE_LAMBDA {
                rbw_stage<C>(a, t, a.x, xdst, nsx, ox, wave, tile, rx);
                rbw_stage<C>(a, t, a.dy, kdst, nsk, ok, wave, tile, 0);
                const int n1 = TH + 2 * ho;
                for (int grp = rw; grp * 16 < t.nsegt * cols; grp += NS) {
                    const WalkAnchor an = walk_anchor(grp * 16 + r16, cols, W, t.nsegt, R, n1, t.inv_c, t.inv_W);
                    uint32_t ta = uint32_t(an.fi * xpf + (an.row0 + 1 - ho) * TW + an.c + 1) * 32 + g * 8;
                    const int hb = h0 - ho + an.row0;   // image row of the walk's first row
                    const uint32_t one = 0x00010001u, top = 0x7f807f80u;
                    uint2 mk = make_uint2(0, 0);
                    walk_conv16<R>(dsrc, an.fi * dpf + an.row0 * TW + an.c, g, rowb, wb,
                        [&] { mk = *reinterpret_cast<const uint2*>(tsrc + ta); },
                        [&](int j, const cb_f32x4& acc) {
                            const int h = hb + j;
                            const bool in = uint32_t(h) < uint32_t(H);   // rows off the frame stay zero
                            uint2 u = make_uint2(pos_mask16x2(mk.x, pack2bf(acc[0], acc[1]), one, top), pos_mask16x2(mk.y, pack2bf(acc[2], acc[3]), one, top));
                            if (!in) u = make_uint2(0, 0);
                            if (an.ok && an.row0 + j >= an.rbeg) *reinterpret_cast<uint2*>(dtdst + ta) = u;
                            ta += rowb;
                        });
                }
            };
            phase_a(xw, skw, dtw, dyw, tw);
            rbw_landed<G::MAXX>(xw, nsx, wave, lane);
            lds_barrier();   // the dt window is complete, x has landed
            auto phase_b = [&](unsigned char* __restrict__ ddst, unsigned char* __restrict__ tdst, const unsigned char* __restrict__ dtsrc,
                               const unsigned char* __restrict__ xsrc, const unsigned char* __restrict__ ksrc) CB_INLINE_LAMBDA {
                if (tile + G0 < t.ntiles) {
                    rbw_stage<C>(a, t, a.dy, ddst, nsd, od, wave, tile + G0, rd);
                    rbw_stage<C>(a, t, a.t, tdst, nsx, ox, wave, tile + G0, rx);
                }
                uint16_t* dxb = static_cast<uint16_t*>(a.dx) + fo;
                for (int grp = rw; grp * 16 < t.nsegx * cols; grp += NS) {
                    const WalkAnchor an = walk_anchor(grp * 16 + r16, cols, W, t.nsegx, R, TH, t.inv_c, t.inv_W);
                    uint32_t xa = uint32_t(an.fi * xpf + (an.row0 + 1) * TW + an.c + 1) * 32 + g * 8;
                    uint32_t ka = uint32_t((an.fi * TH + an.row0) * W + an.c) * 32 + g * 8;
                    uint32_t go = uint32_t(((an.fi * H + h0 + an.row0) * W + an.c) * C + g * 4);
                    const bool own = an.ok && an.fi < nf;
                    uint2 mk = make_uint2(0, 0), sk = make_uint2(0, 0);
                    walk_conv16<R>(dtsrc, an.fi * xpf + an.row0 * TW + an.c, g, rowb, wa,
                        [&] {
                            mk = *reinterpret_cast<const uint2*>(xsrc + xa);
                            sk = *reinterpret_cast<const uint2*>(ksrc + ka);
                            xa += rowb;
                            ka += W * 32;
                        },
                        [&](int j, const cb_f32x4& acc) {
                            if (own && an.row0 + j >= an.rbeg && an.row0 + j < the)
                                store4(dxb + go, (bf_lo(mk.x) > 0.f ? acc[0] : 0.f) + bf_lo(sk.x), (bf_hi(mk.x) > 0.f ? acc[1] : 0.f) + bf_hi(sk.x),
                                       (bf_lo(mk.y) > 0.f ? acc[2] : 0.f) + bf_lo(sk.y), (bf_hi(mk.y) > 0.f ? acc[3] : 0.f) + bf_hi(sk.y));
                            go += W * C;
                        });
                }
            };
            phase_b(dyw, tw, dtw, xw, skw);
        }
        lds_barrier();   // (the weight-gradient role's two barriers)
        lds_barrier();
        return;
    }

    // ---- weight-gradient role: channel blocks (co, ci) of this wave
    lds_barrier();
    clear_dt();
    cb_f32x4 accA[9], accB[9], biasA, biasB;
#pragma unroll
    for (int k = 0; k < 9; ++k) accA[k] = accB[k] = cb_f32x4{0.f, 0.f, 0.f, 0.f};
    biasA = biasB = cb_f32x4{0.f, 0.f, 0.f, 0.f};
    // dwin's own row 0 is window row drow; xwin's row 0 is one image row above it
    auto wgrad = [&](const unsigned char* xwin, const unsigned char* dwin, int dstride, int drow, cb_f32x4 (&acc)[9], cb_f32x4& accb) CB_INLINE_LAMBDA {
        for (int grp = rw; grp * 32 < t.nsegw * cols; grp += NS) {
            int ln = lane;
            asm volatile("" : "+v"(ln));   // (as above)
            const int g = ln >> 4, jj = (ln >> 2) & 3, m = ln & 3;
            int px[2], pd[2], skip[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const WalkAnchor an = walk_anchor(grp * 32 + h * 16 + 4 * g + jj, cols, W, t.nsegw, R, TH, t.inv_c, t.inv_W);
                px[h] = an.fi * xpf + an.row0 * TW + an.c;
                pd[h] = an.fi * dstride + (an.row0 + drow) * TW + an.c + 1;
                skip[h] = an.ok ? an.rbeg - an.row0 : R;
            }
            walk_wgrad16<R>(xwin, dwin, px, pd, skip, uint32_t(m * 8), rowb, acc, accb);
        }
    };
    auto phase_a = [&](unsigned char* __restrict__ xdst, unsigned char* __restrict__ kdst, const unsigned char* __restrict__ tsrc,
                       const unsigned char* __restrict__ dsrc, int tile) CB_INLINE_LAMBDA {
        rbw_stage<C>(a, t, a.x, xdst, nsx, ox, wave, tile, rx);
        rbw_stage<C>(a, t, a.dy, kdst, nsk, ok, wave, tile, 0);
        wgrad(tsrc, dsrc, dpf, 1 + ho, accB, biasB);
    };
    auto phase_b = [&](unsigned char* __restrict__ ddst, unsigned char* __restrict__ tdst, const unsigned char* __restrict__ xsrc,
                       const unsigned char* __restrict__ dtsrc, int next) CB_INLINE_LAMBDA {
        if (next < t.ntiles) {
            rbw_stage<C>(a, t, a.dy, ddst, nsd, od, wave, next, rd);
            rbw_stage<C>(a, t, a.t, tdst, nsx, ox, wave, next, rx);
        }
        wgrad(xsrc, dtsrc, xpf, 1, accA, biasA);
    };
    for (int tile = lg; tile < t.ntiles; tile += G0) {
        rbw_landed<G::MAXX>(tw, nsx, wave, lane);
        lds_barrier();
        phase_a(xw, skw, tw, dyw, tile);
        rbw_landed<G::MAXX>(xw, nsx, wave, lane);
        lds_barrier();
        phase_b(dyw, tw, xw, dtw, tile + G0);
    }

    // ---- the four waves' sums, wave 0 first, through LDS (the dgrad waves are done with it at the
    // barrier), as this workgroup's partials: conv_b's set, then conv_a's
    lds_barrier();
    float* red = reinterpret_cast<float*>(smem);
    const int g = lane >> 4, r16 = lane & 15;
    auto put = [&](int at, const cb_f32x4& acc) {
#pragma unroll
        for (int e = 0; e < 4; ++e) red[(rw * 20 + at) * 256 + (4 * g + e) * 16 + r16] = acc[e];
    };
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        put(k, accB[k]);
        put(10 + k, accA[k]);
    }
    put(9, biasB);
    put(19, biasA);
    lds_barrier();
    float* part = a.partial + int64_t(blockIdx.x) * G::PSTRIDE;
    for (int e = tid - NS * 64; e < 20 * 256; e += NS * 64) {
        const float v = ((red[e] + red[20 * 256 + e]) + red[40 * 256 + e]) + red[60 * 256 + e];
        part[e < 10 * 256 ? e : e - 10 * 256 + t.pset] = v;
    }
}

namespace {

// Scratch: both partial sets. The kernels use one partial per CU at most (256).
constexpr size_t kRbwPartBytes = 24u << 20;

template <class G>
constexpr size_t rbw_partial_floats() {
    const size_t cap = kRbwPartBytes / (2 * size_t(G::PSTRIDE) * sizeof(float));
    return 2 * (cap < 256 ? 256 : (cap > 1024 ? 1024 : cap)) * size_t(G::PSTRIDE);
}

// Launches kernel(std::integral_constant<int, R>) on the tile shape that walkplan.h chooses.
template <class G, class Launch>
hipError_t rbw_launch(const ResBwdArgs& a, hipStream_t s, PendingReduce out[2], Launch&& launch) {
    const int H = a.H, W = a.W, cus = std::min(device_cus(), 256);
    if (int64_t(H) * W * G::C * 2 >= (int64_t(1) << 31)) return hipErrorInvalidValue;
    static thread_local WalkPlans<RbwTile> plans;
    const auto* plan = plans.find(a.n, H, W, cus);
    if (!plan) {
        const size_t limit = std::min<size_t>(lds_limit(), 160 * 1024);
        RbwTile t{};
        size_t L = 0;
        if (!walk_choose([&](auto&& f) { rbw_shapes<G>(a.n, H, W, cus, limit, f); }, t, L)) return hipErrorInvalidValue;
        plan = plans.put({a.n, H, W, cus, t, L});
    }
    const int parts = plan->t.pset / G::PSTRIDE;
    walk_dispatch<G::MAXR>(plan->t.R, [&](auto r) {
        ProfScope ps(s, [&] { return cb_key("resblock_bwd", 0, cb_dims(G::C, G::C) + "/" + cb_dims(H, W)); });
        launch(r, dim3(unsigned(parts)), dim3(G::NT), plan->lds, plan->t);
    });
    out[0] = PendingReduce{a.partial, a.dwb, a.dbb, parts, G::PSTRIDE, G::C, G::C, 0, 1.f};
    out[1] = PendingReduce{a.partial + plan->t.pset, a.dwa, a.dba, parts, G::PSTRIDE, G::C, G::C, 0, 1.f};
    return hipGetLastError();
}

}  // namespace

bool resblock_bwd_supported(int C) { return C == 16 || C == 32; }

// The block backward beats the two conv backward launches at every shape the networks use (32
// channels, 2048 frames: 11x11 45 against 75 us, 21x21 101 against 148 us; 8192 frames at 42x42:
// 1.49 against 1.97 ms).
bool resblock_bwd_preferred(int C, int H, int W) { return (C == 16 || C == 32) && H > 0 && W > 0; }

size_t resblock_bwd_partial_floats(int C) {
    if (C == 16) return rbw_partial_floats<Rbw16Geom>();
    if (C == 32) return rbw_partial_floats<RbwGeom>();
    return 0;
}

hipError_t resblock_bwd(int C, const ResBwdArgs& a, hipStream_t s, PendingReduce out[2]) {
    out[0].nparts = 0;
    out[1].nparts = 0;
    if (a.n <= 0) {
        return flush_pending_reduces(a.pend, a.pend2, s);
    }
    if (C == 16)
        return rbw_launch<Rbw16Geom>(a, s, out, [&](auto r, dim3 grid, dim3 block, size_t lds, const RbwTile& t) {
            hipLaunchKernelGGL(resblock_bwd16_walk_kernel<decltype(r)::value>, grid, block, lds, s, a, t);
        });
    if (C == 32)
        return rbw_launch<RbwGeom>(a, s, out, [&](auto r, dim3 grid, dim3 block, size_t lds, const RbwTile& t) {
            hipLaunchKernelGGL(resblock_bwd_walk_kernel<decltype(r)::value>, grid, block, lds, s, a, t);
        });
    return hipErrorInvalidValue;
}

}  // namespace cb
