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

// The 32-channel block backward by column walks (walk.h), in one 8-wave workgroup per CU with
// two wave roles. Waves 0-3 form dt, then dx, for both channel blocks (both convolutions' weights:
// 144 registers; each input fragment feeds 18 MFMAs); waves 4-7 form conv_b's weight gradient
// while dt is formed and conv_a's beside dx, each wave one 16x16 channel block of all nine taps (18
// tap tiles and the bias columns: 80 registers; each x fragment feeds three rows of dy). A tile (F
// whole frames, or a band of one; walkplan.h) has two phases:
//   a: dt = conv_b^T(dy) * [t > 0] into the dt window; dWb from dy and t; x and dy's own pixels
//      once more (for the skip term) are being staged;
//   b: dx = conv_a^T(dt) * [x > 0] + dy; dWa from dt and x; the next tile's dy and t are staged.
// No phase reads what is being staged in it, so one set of windows in LDS is enough for loads to be in
// flight during all of the work.
// Measured against a form that read every fragment once per tap and block (its own two roles
// bound by LDS and by the vector instructions beside the MFMAs), with the reduce, graph replays on one
// card: 2048 frames of 21x21 128 -> 87 us, of 11x11 56 -> 41, 8192 of 42x42 1637 -> 1469, 640 of 11x11 36 ->
// 27, 128 of 11x11 26 -> 18.
// Counters at 2048 frames of 21x21: 252 MB move where 231 have to (a third of dy's second reads miss the
// L2), the matrix cores are busy 0.33 of the time. What bounds it: a SIMD's MFMAs (about 270 of 16 cycles
// per phase) and the vector instructions of its two waves, and the loads of a phase, which add up with its
// work (walkplan.h); then barriers.
template <int R, bool HELP>
__global__ __launch_bounds__(RbwGeom::NT, 2) void resblock_bwd_walk_kernel(ResBwdArgs a, RbwTile t) {
    using G = RbwGeom;
    constexpr int NT = G::NT, NW = G::NW, NS = G::NS, C = G::C;
    extern __shared__ __align__(16) unsigned char smem[];
    if (HELP && pending_helper<NT>(a, t.pset / G::PSTRIDE, smem)) return;
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
    const unsigned nwg = HELP ? t.pset / G::PSTRIDE : gridDim.x;   // workgroups with tiles
    if ((nwg & 7) == 0) lg = (blockIdx.x & 7) * (nwg >> 3) + (blockIdx.x >> 3);
    const int G0 = int(nwg);

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
    if constexpr (!HELP) {
        if (a.pend.nparts > 0) pending_reduce<NT>(a.pend, dtw);
        if (a.pend2.nparts > 0) pending_reduce<NT>(a.pend2, dtw);
    }
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
// Measured against the tile-by-tile form below, with the reduce, graph replays on one card: 2048 frames of
// 42x42 157 -> 146 us, 640 of 42x42 60 -> 52, of 21x21 35 -> 25, of 11x11 26.5 -> 16.7, 8192 of 21x21 150 -> 136.
// Two workgroups of this form per CU (80 KB windows, 128 registers, which spill) were slower. What bounds it:
// 462 MB (468 move) at the rate of a large copy are 97 us; the rest is work and loads of a phase that add up,
// and barriers.
template <int R, bool HELP>
__global__ __launch_bounds__(Rbw16Geom::NT, 2) void resblock_bwd16_walk_kernel(ResBwdArgs a, RbwTile t) {
    using G = Rbw16Geom;
    constexpr int NT = G::NT, NW = G::NW, NS = G::NS, C = G::C;
    extern __shared__ __align__(16) unsigned char smem[];
    if (HELP && pending_helper<NT>(a, t.pset / G::PSTRIDE, smem)) return;
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
    const unsigned nwg = HELP ? t.pset / G::PSTRIDE : gridDim.x;   // workgroups with tiles
    if ((nwg & 7) == 0) lg = (blockIdx.x & 7) * (nwg >> 3) + (blockIdx.x >> 3);
    const int G0 = int(nwg);

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
    if constexpr (!HELP) {
        if (a.pend.nparts > 0) pending_reduce<NT>(a.pend, dtw);
        if (a.pend2.nparts > 0) pending_reduce<NT>(a.pend2, dtw);
    }
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

// The 16-channel block backward tile by tile, two workgroups per CU: a tile is a band of TH rows of one
// frame, staged whole (dy on rows h0-2 .. h0+TH+1, t and x on rows h0-1 .. h0+TH), and all waves take
// each phase's 16-pixel column tiles in turn. It reads every fragment once per tap, waits for its
// loads and meets four barriers per tile, all of which the other workgroup overlaps, but its work
// falls evenly on the waves whatever the width, where the walks pay for whole groups of 16 columns and
// whole segments of rows. Walks against tiles, in turn on one card: 2048 frames of 42x42 144 against 155
// us, 8192 of 21x21 134 against 152; but 8192 of 30x45 469 against 411, 32x32 347 against 320, 48x40 614
// against 569, 2048 of 84x84 658 against 593. walkplan.h estimates both and takes the shorter.
__global__ __launch_bounds__(RbtGeom::NT, 4) void resblock_bwd16_tile_kernel(ResBwdArgs a, RbtTile t) {
    using G = RbtGeom;
    constexpr int C = G::C, NW = G::NW, NT = G::NT, PX = G::PX, NB = G::NBB - 1;
    constexpr int KSD = 5;                       // input-gradient k-steps of two taps
    // weight gradients: waves 0 .. 3 form conv_b's, the others conv_a's, each wave TPW column
    // blocks (a tap, or the bias), so each dy / dt fragment is read by half the waves
    constexpr int NWG = NW / 2, TPW = (G::NBB + NWG - 1) / NWG;

    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* zero = smem;                   // 64 zero bytes
    unsigned char* dyw = smem + t.dy_off;         // dy [TH+4][W+2], row 0 = image row h0-2
    unsigned char* tw = smem + t.t_off + PX;      // relu(t) [TH+2][W+2], row 0 = h0-1, guard pixels
    unsigned char* xw = smem + t.x_off + PX;      // relu(x) [TH+2][W+2], likewise
    unsigned char* dtw = smem + t.dt_off;         // dt [TH+2][W+2], row 0 = h0-1

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, r16 = lane & 15, jj = r16 >> 2, m = r16 & 3;
    const int H = a.H, W = a.W, TH = t.TH, TW = W + 2;

    // earlier launches' weight-gradient partials, summed first (LDS is free until staging)
    if (a.pend.nparts > 0) pending_reduce<NT>(a.pend, smem);
    if (a.pend2.nparts > 0) pending_reduce<NT>(a.pend2, smem);
    if (tid < 16) reinterpret_cast<uint32_t*>(zero)[tid] = 0u;
    // the dt window: its padding columns are never written
    for (int j = tid; j < t.dt_bytes / 16; j += NT) reinterpret_cast<uint4*>(dtw)[j] = make_uint4(0, 0, 0, 0);
    // the t and x windows' guard pixels (read only against zero dy / dt, never staged)
    if (tid < PX / 4) {
        reinterpret_cast<uint32_t*>(tw - PX)[tid] = 0u;
        reinterpret_cast<uint32_t*>(tw + t.tx_guard)[tid] = 0u;
        reinterpret_cast<uint32_t*>(xw - PX)[tid] = 0u;
        reinterpret_cast<uint32_t*>(xw + t.tx_guard)[tid] = 0u;
    }

    // ---- input-gradient A fragments of both convs: A[o][k] = w[8 - tap][o][co] with k = tap * 16 + co
    // (zero past the 9 taps; loads clamped)
    const int ci0 = g * 4;   // the lane's first output channel
    uint4 wfa[KSD], wfb[KSD];
    auto load_w = [&](const float* w, uint4 (&wf)[KSD]) CB_INLINE_LAMBDA {
#pragma unroll
        for (int ks = 0; ks < KSD; ++ks) {
            const int tap = 2 * ks + (g >> 1);
            const float* p = w + ((tap < 9 ? 8 - tap : 0) * C + r16) * C + (g & 1) * 8;
            const float4 u = load_f4(p), v = load_f4(p + 4);
            wf[ks] = make_uint4(pack2bf(u.x, u.y), pack2bf(u.z, u.w), pack2bf(v.x, v.y), pack2bf(v.z, v.w));
            if (tap >= 9) wf[ks] = make_uint4(0, 0, 0, 0);
        }
    };
    load_w(a.wa, wfa);
    load_w(a.wb, wfb);
    // B-fragment byte offsets from the lane's tap-(0,0) pixel of a dy-like window: a k-step spans
    // two taps; past the ninth the lanes read the zero bytes (an infinite value times a zero weight
    // would be NaN)
    int dboff[KSD];
#pragma unroll
    for (int ks = 0; ks < KSD; ++ks) {
        const int tap = 2 * ks + (g >> 1);
        dboff[ks] = ((tap / 3) * TW + tap % 3) * PX + (g & 1) * 16;
    }
    auto dgrad = [&](const uint4 (&wf)[KSD], const unsigned char* xb) CB_INLINE_LAMBDA {
        cb_f32x4 acc = cb_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KSD; ++ks) {
            const unsigned char* p = ks == KSD - 1 && g >= 2 ? zero : xb + dboff[ks];
            acc = PrecBF16::mma(wf[ks], *reinterpret_cast<const uint4*>(p), acc);
        }
        return acc;
    };
    // weight-gradient column blocks nb = wg + NWG * i (one tap, or the bias block) of conv_b
    // (grp 0) or conv_a (grp 1)
    const int wg = wave % NWG, grp = wave / NWG;
    int wboff[TPW];
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
        const int nb = wg + NWG * i;
        wboff[i] = nb < NB ? ((nb / 3) * TW + nb % 3) * PX + 8 * m : 0;
    }
    cb_f32x4 wacc[TPW];
#pragma unroll
    for (int i = 0; i < TPW; ++i) wacc[i] = cb_f32x4{0.f, 0.f, 0.f, 0.f};
    const uint4 ones = make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);

    // ---- staging offsets, tile-invariant per lane (slot k of this wave: j = (wave + NW*k)*64
    // + lane: pixel j / 2, half j % 2), relative to the window's first row at image row 0; a tile
    // adds that row's image row. Rows off the frame fall outside the frame's buffer resource and
    // read zero, as do padding columns (kOOB).
    const int nsd = (TH + 4) * TW * 2, nsx = (TH + 2) * TW * 2;
    auto win_off = [&](int j, int ns) CB_INLINE_LAMBDA {
        const int p = j >> 1, rr = qdiv(p, t.inv_TW), col = p - rr * TW;
        const uint32_t off = uint32_t(((rr * W + col - 1) * C + (j & 1) * 8) * 2);
        return (j < ns) & (uint32_t(col - 1) < uint32_t(W)) ? off : kOOB;
    };
    uint32_t od[G::MAXS], ox[G::MAXS];
#pragma unroll
    for (int k = 0; k < G::MAXS; ++k) {
        od[k] = win_off((wave + NW * k) * 64 + lane, nsd);
        ox[k] = win_off((wave + NW * k) * 64 + lane, nsx);
    }

    // ---- one weight gradient over the band's own rows: dy-like window dwin (own row 0 at
    // window row drow0) against the relu'd window bwin (row 0 = image row h0-1): pixel idx of
    // the own rows pairs with bwin pixel idx - 1 + tap offset. Lane (g, 4jj+m) takes pixels
    // o = 16*half + 4g + jj (channels 4m ..).
    auto wgrad = [&](const unsigned char* dwin, int drow0, const unsigned char* bwin, const unsigned char* bguard, int L) {
        // specialised per wave, so that each column block's kind (loaded or bias) is known at
        // compile time and the k-step loop carries no branches
        auto run = [&](auto wv) {
            constexpr int WG = decltype(wv)::value;
            const int nfull = L >> 5, o0 = 4 * g + jj;
            const unsigned char* ap = dwin + (drow0 * TW + o0) * PX + 8 * m;
            const unsigned char* bp = bwin + (o0 - 1) * PX;
            auto kstep = [&](const unsigned char* a0, const unsigned char* a1, const unsigned char* b0, const unsigned char* b1) {
                const uint2 alo = lds_read_tr16(a0), ahi = lds_read_tr16(a1);   // a0, a1: zero past L
                const uint4 af = make_uint4(alo.x, alo.y, ahi.x, ahi.y);
#pragma unroll
                for (int i = 0; i < TPW; ++i) {
                    const int nb = WG + NWG * i;
                    if (nb < NB) {
                        const uint2 lo = lds_read_tr16(b0 + wboff[i]), hi = lds_read_tr16(b1 + wboff[i]);
                        wacc[i] = PrecBF16::mma(af, make_uint4(lo.x, lo.y, hi.x, hi.y), wacc[i]);
                    } else if (nb == NB) {   // the bias block: a column of ones
                        wacc[i] = PrecBF16::mma(af, ones, wacc[i]);
                    }
                }
            };
            int ks = 0;
            for (; ks + 2 <= nfull; ks += 2) {   // two k-steps per trip: half the pointer updates
                kstep(ap, ap + 16 * PX, bp, bp + 16 * PX);
                kstep(ap + 32 * PX, ap + 48 * PX, bp + 32 * PX, bp + 48 * PX);
                ap += 64 * PX;
                bp += 64 * PX;
            }
            if (ks < nfull) {
                kstep(ap, ap + 16 * PX, bp, bp + 16 * PX);
                ap += 32 * PX;
                bp += 32 * PX;
            }
            if (L & 31) {   // the last, partial k-step
                const int o = nfull * 32 + o0;
                const bool ok0 = o < L, ok1 = o + 16 < L;
                kstep(ok0 ? ap : zero, ok1 ? ap + 16 * PX : zero, ok0 ? bp : bguard, ok1 ? bp + 16 * PX : bguard);
            }
        };
        static_assert(NWG == 4, "one specialisation per wave of a group");
        switch (wg) {
            case 0: run(std::integral_constant<int, 0>{}); break;
            case 1: run(std::integral_constant<int, 1>{}); break;
            case 2: run(std::integral_constant<int, 2>{}); break;
            default: run(std::integral_constant<int, 3>{}); break;
        }
    };

    int lg = blockIdx.x;   // neighbouring bands (which share halo rows) on one XCD
    if ((gridDim.x & 7) == 0) lg = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);

    for (int tile = lg; tile < t.ntiles; tile += gridDim.x) {
        const int band = tile % t.nbands, f = tile / t.nbands;
        const int h0 = band * TH, the = H - h0 < TH ? H - h0 : TH;
        const int64_t fo = int64_t(f) * H * W * C;   // the frame's first element
        __syncthreads();   // the previous tile's LDS reads are done

        // ---- stage dy (rows h0-2 ..), t and x (rows h0-1 ..)
        {
            const uint32_t fb = uint32_t(H) * W * C * 2;
            const auto rd = buf_rsrc(static_cast<const uint16_t*>(a.dy) + fo, fb);
            const auto rt = buf_rsrc(static_cast<const uint16_t*>(a.t) + fo, fb);
            const auto rx = buf_rsrc(static_cast<const uint16_t*>(a.x) + fo, fb);
            const uint32_t hd = uint32_t((h0 - 2) * W * C * 2);   // wraps above the frame: reads zero
            const uint32_t hx = uint32_t((h0 - 1) * W * C * 2);
#pragma unroll
            for (int k = 0; k < G::MAXS; ++k)
                if ((wave + NW * k) * 64 < nsd) dma16_to_lds(rd, dyw + (wave + NW * k) * 1024, od[k] + hd);
#pragma unroll
            for (int k = 0; k < G::MAXS; ++k)
                if ((wave + NW * k) * 64 < nsx) {
                    dma16_to_lds(rt, tw + (wave + NW * k) * 1024, ox[k] + hx);
                    dma16_to_lds(rx, xw + (wave + NW * k) * 1024, ox[k] + hx);
                }
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        {
            // both convs read relu'd inputs; relu(v) > 0 exactly where v > 0, so the masks
            // read the same windows
            uint4* t4 = reinterpret_cast<uint4*>(tw);
            uint4* x4 = reinterpret_cast<uint4*>(xw);
            for (int j = tid; j < nsx; j += NT) {
                const uint4 u = t4[j], v = x4[j];
                t4[j] = relu8(u);
                x4[j] = relu8(v);
            }
        }
        __syncthreads();

        // ---- conv_b's input gradient dt on window rows r = 0 .. the+1 (image rows h0-1+r;
        // zero off the frame), 16-pixel column tiles, into the dt window
        {
            const int npx = (the + 2) * W;
            for (int nt = wave; nt * 16 < npx; nt += NW) {
                const int q = nt * 16 + r16;
                const int qc = q < npx ? q : npx - 1;   // past npx: computed, not stored
                const int row = qdiv(qc, t.inv_W), col = qc - row * W;
                const unsigned char* xb = dyw + (row * TW + col) * PX;
                const cb_f32x4 acc = dgrad(wfb, xb);
                if (q < npx) {
                    const int h = h0 - 1 + row;
                    uint2 o = make_uint2(0u, 0u);
                    if (h >= 0 && h < H) {
                        float mk[4];
                        load4(reinterpret_cast<const uint16_t*>(tw + (row * TW + col + 1) * PX + ci0 * 2), mk);
                        o = make_uint2(pack2bf(mk[0] > 0.f ? acc[0] : 0.f, mk[1] > 0.f ? acc[1] : 0.f),
                                       pack2bf(mk[2] > 0.f ? acc[2] : 0.f, mk[3] > 0.f ? acc[3] : 0.f));
                    }
                    *reinterpret_cast<uint2*>(dtw + (row * TW + col + 1) * PX + ci0 * 2) = o;
                }
            }
        }
        __syncthreads();   // the dt window is complete

        // ---- dx = conv_a^T(dt) * [x > 0] + dy on the band's rows
        {
            const int npx = the * W;
            uint16_t* dxt = static_cast<uint16_t*>(a.dx) + fo + int64_t(h0) * W * C;
            for (int nt = wave; nt * 16 < npx; nt += NW) {
                const int q = nt * 16 + r16;
                const int qc = q < npx ? q : npx - 1;
                const int row = qdiv(qc, t.inv_W), col = qc - row * W;
                const unsigned char* xb = dtw + (row * TW + col) * PX;
                const cb_f32x4 acc = dgrad(wfa, xb);
                if (q < npx) {
                    float mk[4], sk[4];
                    load4(reinterpret_cast<const uint16_t*>(xw + ((row + 1) * TW + col + 1) * PX + ci0 * 2), mk);
                    load4(reinterpret_cast<const uint16_t*>(dyw + ((row + 2) * TW + col + 1) * PX + ci0 * 2), sk);
                    float v[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[j] = (mk[j] > 0.f ? acc[j] : 0.f) + sk[j];
                    store4(dxt + uint32_t(q * C + ci0), v[0], v[1], v[2], v[3]);
                }
            }
        }
        // ---- the weight gradients: conv_b's, dy (own rows from dy-window row 2) against
        // relu(t), by the first half of the waves; conv_a's, dt (own rows from dt-window row
        // 1) against relu(x), by the second
        if (grp == 0) wgrad(dyw, 2, tw, tw - PX, the * TW);
        else wgrad(dtw, 1, xw, xw - PX, the * TW);
    }

    // ---- this workgroup's partials: conv_b's set, then conv_a's, each [nb][co 16][ci 16]
    float* part = a.partial + (grp == 0 ? 0 : t.pset) + int64_t(blockIdx.x) * G::PSTRIDE;
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
        const int nb = wg + NWG * i;
        if (nb < G::NBB)
#pragma unroll
            for (int e = 0; e < 4; ++e) part[nb * 256 + (4 * g + e) * 16 + r16] = wacc[i][e];
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

void rbw_pending(const ResBwdArgs& a, int C, int parts, int pstride, int pset, PendingReduce out[2]) {
    out[0] = PendingReduce{a.partial, a.dwb, a.dbb, parts, pstride, C, C, 0, 1.f};
    out[1] = PendingReduce{a.partial + pset, a.dwa, a.dba, parts, pstride, C, C, 0, 1.f};
}

hipError_t rb32_launch(const ResBwdArgs& a, hipStream_t s, PendingReduce out[2]) {
    using G = RbwGeom;
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
    const int parts = plan->t.pset / G::PSTRIDE, helpers = pending_helpers(a, parts, cus);
    walk_dispatch<G::MAXR>(plan->t.R, [&](auto r) {
        ProfScope ps(s, [&] { return cb_key("resblock_bwd", 0, cb_dims(G::C, G::C) + "/" + cb_dims(H, W)); });
        const auto kernel = helpers ? resblock_bwd_walk_kernel<decltype(r)::value, true> : resblock_bwd_walk_kernel<decltype(r)::value, false>;
        hipLaunchKernelGGL(kernel, dim3(unsigned(parts + helpers)), dim3(G::NT), plan->lds, s, a, plan->t);
    });
    rbw_pending(a, G::C, parts, G::PSTRIDE, plan->t.pset, out);
    return hipGetLastError();
}

hipError_t rb16_launch(const ResBwdArgs& a, hipStream_t s, PendingReduce out[2]) {
    using G = Rbw16Geom;
    const int H = a.H, W = a.W, cus = std::min(device_cus(), 256);
    if (int64_t(H) * W * G::C * 2 >= (int64_t(1) << 31)) return hipErrorInvalidValue;
    static thread_local WalkPlans<Rb16Plan> plans;
    const auto* plan = plans.find(a.n, H, W, cus);
    if (!plan) {
        const size_t limit = std::min<size_t>(lds_limit(), 160 * 1024);
        Rb16Plan p{};
        size_t L = 0;
        if (!rb16_choose(a.n, H, W, cus, limit, p, L)) return hipErrorInvalidValue;
        if (p.tiles) {
            const void* fn = reinterpret_cast<const void*>(&resblock_bwd16_tile_kernel);
            const int room = int(resblock_bwd_partial_floats(G::C) / (2 * size_t(G::PSTRIDE)));
            p.u.pset = std::min({std::max(1, resident_blocks(fn, RbtGeom::NT, L)), room, p.u.ntiles}) * G::PSTRIDE;
        }
        plan = plans.put({a.n, H, W, cus, p, L});
    }
    const Rb16Plan& p = plan->t;
    const int pset = p.tiles ? p.u.pset : p.t.pset, parts = pset / G::PSTRIDE;
    auto scope = [&] { return cb_key("resblock_bwd", 0, cb_dims(G::C, G::C) + "/" + cb_dims(H, W)); };
    if (p.tiles) {
        ProfScope ps(s, scope);
        hipLaunchKernelGGL(resblock_bwd16_tile_kernel, dim3(unsigned(parts)), dim3(RbtGeom::NT), plan->lds, s, a, p.u);
    } else {
        const int helpers = pending_helpers(a, parts, cus);   // (tiles are taken one by one only where they are many)
        walk_dispatch<G::MAXR>(p.t.R, [&](auto r) {
            ProfScope ps(s, scope);
            const auto kernel = helpers ? resblock_bwd16_walk_kernel<decltype(r)::value, true> : resblock_bwd16_walk_kernel<decltype(r)::value, false>;
            hipLaunchKernelGGL(kernel, dim3(unsigned(parts + helpers)), dim3(G::NT), plan->lds, s, a, p.t);
        });
    }
    rbw_pending(a, G::C, parts, G::PSTRIDE, pset, out);
    return hipGetLastError();
}

}  // namespace

bool resblock_bwd_supported(int C) { return C == 16 || C == 32; }

// The block backward beats the two conv backward launches at every shape the networks use (32
// channels, 2048 frames: 11x11 41 against 75 us, 21x21 87 against 148 us; 8192 frames at 42x42:
// 1.47 against 1.97 ms).
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
    if (C == 16) return rb16_launch(a, s, out);
    if (C == 32) return rb32_launch(a, s, out);
    return hipErrorInvalidValue;
}

}  // namespace cb
