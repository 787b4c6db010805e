// Column walks: 3x3 convolutions of 16, 32 and 64 channels, and their weight gradients, over LDS windows, with
// every fragment read feeding all the rows it touches.
//
// The windows (walkplan.h) hold rows of W + 1 pixels: column 0 is zero padding, the right
// neighbour of a row's last pixel the next row's column 0. A pixel's 32 channels take 64 bytes,
// its four 16-byte slots permuted by XOR with 2 * bit 2 of its column: 16-byte reads of 16
// consecutive pixels, and 8-byte transpose reads of 8, then fall on distinct banks, and a step of
// one row is one constant. A group of anchors that goes on in the next segment or frame (every group of
// an 11-column frame, half of a 21-column one's) jumps in between and folds some of its reads onto one
// bank: 0.26 to 0.53 of the LDS-active cycles are conflicts (21x21 backward, 11x11 forward).
//
// The pixels of a fragment are anchors: a column of the tile, or one of nseg segments of it, R
// rows each. All lanes walk down their anchors together.
#pragma once

#include <type_traits>

#include "common.h"
#include "walkplan.h"

namespace cb {

// Byte offset, in a pixel's 64 bytes at window column col, of the 16-byte slot or 8-byte chunk that
// starts at channel byte ch.
CB_DEV uint32_t walk_ch(uint32_t col, uint32_t ch) { return ch ^ ((col << 3) & 32); }

// Anchor `id` of nseg * cols (cols = F * W): frame fi, column c, rows [row0, row0 + R) of nrows. The
// last segment starts early enough to end at nrows; its rows below rbeg belong to the one above.
struct WalkAnchor { int row0, rbeg, fi, c; bool ok; };
CB_DEV WalkAnchor walk_anchor(int id, int cols, int W, int nseg, int R, int nrows, float inv_c, float inv_W) {
    WalkAnchor an;
    const int last = nseg * cols - 1, ic = id < last ? id : last;
    const int s = qdiv(ic, inv_c), rem = ic - s * cols;
    an.fi = qdiv(rem, inv_W);
    an.c = rem - an.fi * W;
    an.rbeg = s * R;
    an.row0 = s * R < nrows - R ? s * R : nrows - R;
    an.ok = id <= last;
    return an;
}

// Calls f(std::integral_constant<int, R>) for a run-time R of 1 .. MAXR.
template <int MAXR, int R0 = 1, class F>
inline void walk_dispatch(int R, F&& f) {
    if (R == R0) f(std::integral_constant<int, R0>{});
    else if constexpr (R0 < MAXR) walk_dispatch<MAXR, R0 + 1>(R, f);
}
template <class A>
inline int pending_helpers(const A& a, int parts, int room) {
    const int blocks = (a.pend.nparts > 0 ? a.pend.pstride / 64 : 0) + (a.pend2.nparts > 0 ? a.pend2.pstride / 64 : 0);
    return pend_helpers(blocks, parts, room);
}

// The last tile shapes chosen, per thread (the choice takes some microseconds): a few entries by
// problem size, overwritten in turn.
template <class Tile>
struct WalkPlans {
    struct Entry { int64_t n; int H, W, cus; Tile t; size_t lds; };
    Entry e[8];
    int used = 0, next = 0;
    const Entry* find(int64_t n, int H, int W, int cus) const {
        for (int i = 0; i < used; ++i)
            if (e[i].n == n && e[i].H == H && e[i].W == W && e[i].cus == cus) return &e[i];
        return nullptr;
    }
    const Entry* put(const Entry& v) {
        Entry* p = &e[next];
        *p = v;
        next = (next + 1) % 8;
        used = used < 8 ? used + 1 : 8;
        return p;
    }
};

CB_DEV uint4 relu8(uint4 v) {
    return make_uint4(relu_bf16x2(v.x), relu_bf16x2(v.y), relu_bf16x2(v.z), relu_bf16x2(v.w));
}

// One walk of a 3x3 convolution, 32 -> 32 channels: R output rows at the lane's anchor, whose
// tap-(0,0) pixel of the first row is p0, at window column c. w[b][tap] are the A fragments of
// output block b, whose row 4 i + j is channel 8 i + 4 b + j, so that acc[b][j] is channel
// 8 (lane / 16) + 4 b + j. pre() is called before the last MFMAs of each output row, emit(j, acc)
// after them. A wave's vector instructions and MFMAs take turns (4 and 16 cycles each, measured
// to add up within a wave), so nothing is copied: R is a constant and the rows are unrolled, the
// sums of an output row staying in one of three accumulators, input rows alternating between
// two sets of fragment registers.
template <int R, bool RELU, class Pre, class Emit>
CB_DEV void walk_conv32(const unsigned char* win, int p0, int c, int g, int rowb, const uint4 (&w)[2][9], Pre&& pre, Emit&& emit) {
    uint32_t ad[3];
    uint4 x[2][3];
    cb_f32x4 acc[3][2];
    auto load = [&](uint4 (&dst)[3]) CB_INLINE_LAMBDA {
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) dst[kx] = *reinterpret_cast<const uint4*>(win + ad[kx]);
    };
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) ad[kx] = uint32_t(p0 + kx) * 64 + walk_ch(uint32_t(c + kx), uint32_t(g) * 16);
    load(x[0]);
#pragma unroll
    for (int i = 0; i < R + 2; ++i) {   // input row i: tap rows 2, 1, 0 of output rows i - 2, i - 1, i
        uint4 (&cur)[3] = x[i & 1];
        if (i < R + 1) {                // the next row's fragments, in flight during this row's MFMAs
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) ad[kx] += rowb;
            load(x[(i + 1) & 1]);
        }
        if (RELU)
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) cur[kx] = relu8(cur[kx]);
        if (i >= 2) pre();
#pragma unroll
        for (int ky = 2; ky >= 0; --ky)
            if (i >= ky && i - ky < R)
#pragma unroll
                for (int kx = 0; kx < 3; ++kx)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
                        acc[(i - ky) % 3][b] = PrecBF16::mma(w[b][3 * ky + kx], cur[kx],
                                                             ky + kx == 0 ? cb_f32x4{0.f, 0.f, 0.f, 0.f} : acc[(i - ky) % 3][b]);
        if (i >= 2) emit(i - 2, acc[(i - 2) % 3]);
        __builtin_amdgcn_sched_barrier(0);   // one row's reads in flight: registers are short
    }
}

// One walk of a 3x3 weight gradient for one block of 16 input and one of 16 output channels, 64
// anchors as two fragments of 32 (two at once: a step then has MFMAs enough to cover its reads):
// acc[tap][...] += sum over the anchors and R rows of dy[row] (rows of D: output channels) times
// x[row + ky - 1, col + kx - 1] (columns: input channels); accb += sum of dy.
// Lane (g, 4 jj + m) addresses channels 4m .. of anchors 16 h + 4 g + jj, h = 0 .. 3: px[h] is the
// tap-(0,0) pixel of its first row in xwin (window column c[h]), pd[h] that row's pixel in dwin;
// rows below skip[h] add nothing (they read pixel 0 of dwin, which is zero). chx,
// chd: byte of the lane's chunk in a pixel. Each x fragment feeds the three dy rows it meets.
template <int R>
CB_DEV void walk_wgrad(const unsigned char* xwin, const unsigned char* dwin, const int (&px)[4], const int (&pd)[4], const int (&c)[4],
                       const int (&skip)[4], uint32_t chx, uint32_t chd, int rowb, cb_f32x4 (&acc)[9], cb_f32x4& accb) {
    uint32_t ax[4][3], ad[4];
    uint4 x[2][3], d[3][2];
    const uint4 ones = make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
    auto load_d = [&](uint4& dst, int q, int i) CB_INLINE_LAMBDA {
        const uint2 lo = lds_read_tr16(dwin + (i >= skip[2 * q] ? ad[2 * q] : 0u));
        const uint2 hi = lds_read_tr16(dwin + (i >= skip[2 * q + 1] ? ad[2 * q + 1] : 0u));
        dst = make_uint4(lo.x, lo.y, hi.x, hi.y);
    };
    auto load_x = [&](int q) CB_INLINE_LAMBDA {
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) {
            const uint2 lo = lds_read_tr16(xwin + ax[2 * q][kx]), hi = lds_read_tr16(xwin + ax[2 * q + 1][kx]);
            x[q][kx] = make_uint4(lo.x, lo.y, hi.x, hi.y);
        }
    };
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        ad[h] = uint32_t(pd[h]) * 64 + walk_ch(uint32_t(c[h] + 1), chd);
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) ax[h][kx] = uint32_t(px[h] + kx) * 64 + walk_ch(uint32_t(c[h] + kx), chx);
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        load_x(q);
        load_d(d[0][q], q, 0);
    }
    // x row i: tap rows 2, 1, 0 against dy rows i - 2, i - 1, i, row j in d[j % 3]. Each
    // fragment's next rows are read into the registers its MFMAs have just taken, while the
    // other fragment's MFMAs run.
#pragma unroll
    for (int i = 0; i < R + 2; ++i)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
#pragma unroll
            for (int ky = 2; ky >= 0; --ky)
                if (i >= ky && i - ky < R)
#pragma unroll
                    for (int kx = 0; kx < 3; ++kx) acc[3 * ky + kx] = PrecBF16::mma(d[(i - ky) % 3][q], x[q][kx], acc[3 * ky + kx]);
            if (i < R) accb = PrecBF16::mma(d[i % 3][q], ones, accb);
            __builtin_amdgcn_sched_barrier(0);
            if (i < R + 1) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int kx = 0; kx < 3; ++kx) ax[2 * q + h][kx] += rowb;
                load_x(q);
            }
            if (i + 1 < R) {
#pragma unroll
                for (int h = 0; h < 2; ++h) ad[2 * q + h] += rowb;
                load_d(d[(i + 1) % 3][q], q, i + 1);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
}

// ---- 16 channels: 32 bytes per pixel, as they are (16-byte reads of 16 consecutive pixels and
// transpose reads of 8 are free of bank conflicts). A k-step of 32 is two taps, in the order of the
// per-layer kernels: (0,1) (2,3) (4,5) (6,7) (8), the last against zero weights in its second half.

// walk_conv32 for 16 -> 16 channels: w[k-step], output row 4 i + j is channel 4 i + j. Input row i
// serves output rows i (taps 0,1; with row i + 1: 2,3), i - 1 (4,5) and i - 2 (6,7; 8).
template <int R, class Pre, class Emit>
CB_DEV void walk_conv16(const unsigned char* win, int p0, int g, int rowb, const uint4 (&w)[5], Pre&& pre, Emit&& emit) {
    const uint32_t base = uint32_t(p0) * 32 + uint32_t(g & 1) * 16;
    const bool up = g >= 2;
    uint32_t a01 = base + (up ? 32u : 0u), a12 = base + (up ? 64u : 32u), am = up ? base + rowb : base + 64u;
    uint32_t a2 = up ? uint32_t(g & 1) * 16 : base + 64u;
    const uint32_t row2 = up ? 0u : uint32_t(rowb);
    uint4 x[2][4];
    cb_f32x4 acc[3];
    auto load = [&](uint4 (&dst)[4], int i) CB_INLINE_LAMBDA {
        dst[0] = *reinterpret_cast<const uint4*>(win + a01);
        if (i < R) dst[1] = *reinterpret_cast<const uint4*>(win + am);
        if (i >= 1 && i <= R) dst[2] = *reinterpret_cast<const uint4*>(win + a12);
        if (i >= 2) dst[3] = *reinterpret_cast<const uint4*>(win + a2);
    };
    load(x[0], 0);
#pragma unroll
    for (int i = 0; i < R + 2; ++i) {
        const uint4 (&cur)[4] = x[i & 1];
        if (i < R + 1) {
            a01 += rowb; a12 += rowb; am += rowb; a2 += row2;
            load(x[(i + 1) & 1], i + 1);
        }
        if (i >= 2) {
            pre();
            acc[(i - 2) % 3] = PrecBF16::mma(w[3], cur[0], acc[(i - 2) % 3]);
        }
        if (i < R) acc[i % 3] = PrecBF16::mma(w[0], cur[0], cb_f32x4{0.f, 0.f, 0.f, 0.f});
        if (i >= 1 && i <= R) acc[(i - 1) % 3] = PrecBF16::mma(w[2], cur[2], acc[(i - 1) % 3]);
        if (i >= 2) acc[(i - 2) % 3] = PrecBF16::mma(w[4], cur[3], acc[(i - 2) % 3]);
        if (i < R) acc[i % 3] = PrecBF16::mma(w[1], cur[1], acc[i % 3]);
        if (i >= 2) emit(i - 2, acc[(i - 2) % 3]);
        __builtin_amdgcn_sched_barrier(0);   // one row's reads in flight
    }
}

// walk_wgrad for 16 x 16 channels over one fragment of 32 anchors (ch: byte of the lane's chunk).
template <int R>
CB_DEV void walk_wgrad16(const unsigned char* xwin, const unsigned char* dwin, const int (&px)[2], const int (&pd)[2], const int (&skip)[2],
                         uint32_t ch, int rowb, cb_f32x4 (&acc)[9], cb_f32x4& accb) {
    uint32_t ax[2], ad[2];
    uint4 x[2][3], d[4];
    const uint4 ones = make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
    auto load_d = [&](uint4& dst, int i) CB_INLINE_LAMBDA {
        const uint2 lo = lds_read_tr16(dwin + (i >= skip[0] ? ad[0] : 0u)), hi = lds_read_tr16(dwin + (i >= skip[1] ? ad[1] : 0u));
        dst = make_uint4(lo.x, lo.y, hi.x, hi.y);
    };
    auto load_x = [&](uint4 (&dst)[3]) CB_INLINE_LAMBDA {
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) {
            const uint2 lo = lds_read_tr16(xwin + ax[0] + kx * 32), hi = lds_read_tr16(xwin + ax[1] + kx * 32);
            dst[kx] = make_uint4(lo.x, lo.y, hi.x, hi.y);
        }
    };
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        ad[h] = uint32_t(pd[h]) * 32 + ch;
        ax[h] = uint32_t(px[h]) * 32 + ch;
    }
    load_d(d[0], 0);
    load_x(x[0]);
#pragma unroll
    for (int i = 0; i < R + 2; ++i) {
        const uint4 (&cur)[3] = x[i & 1];
        if (i + 1 < R) {
            ad[0] += rowb;
            ad[1] += rowb;
            load_d(d[(i + 1) % 4], i + 1);
        }
        if (i < R + 1) {
            ax[0] += rowb;
            ax[1] += rowb;
            load_x(x[(i + 1) & 1]);
        }
#pragma unroll
        for (int ky = 2; ky >= 0; --ky)
            if (i >= ky && i - ky < R)
#pragma unroll
                for (int kx = 0; kx < 3; ++kx) acc[3 * ky + kx] = PrecBF16::mma(d[(i - ky) % 4], cur[kx], acc[3 * ky + kx]);
        if (i < R) accb = PrecBF16::mma(d[i % 4], ones, accb);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// ---- 64 channels: 128 bytes per pixel, the eight 16-byte slots permuted by XOR with bits 1, 2 of the
// column (free of bank conflicts for the same reads). A fragment's registers take the next row's
// fragment as soon as its MFMAs are issued, so one set of them is enough.
CB_DEV uint32_t walk64_ch(uint32_t col, uint32_t ch) { return ch ^ ((col << 4) & 96); }

// walk_conv32 for 64 input channels and 32 of the output channels: w[b][2 tap + half].
template <int R, class Pre, class Emit>
CB_DEV void walk_conv64(const unsigned char* win, int p0, int c, int g, int rowb, const uint4 (&w)[2][18], Pre&& pre, Emit&& emit) {
    uint32_t ad[3][2];
    uint4 x[3][2];
    cb_f32x4 acc[3][2];
#pragma unroll
    for (int kx = 0; kx < 3; ++kx)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            ad[kx][h] = uint32_t(p0 + kx) * 128 + walk64_ch(uint32_t(c + kx), uint32_t(h) * 64 + uint32_t(g) * 16);
            x[kx][h] = *reinterpret_cast<const uint4*>(win + ad[kx][h]);
        }
#pragma unroll
    for (int i = 0; i < R + 2; ++i) {
        pre(i);
#pragma unroll
        for (int kx = 0; kx < 3; ++kx)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int ky = 2; ky >= 0; --ky)
                    if (i >= ky && i - ky < R)
#pragma unroll
                        for (int b = 0; b < 2; ++b)
                            acc[(i - ky) % 3][b] = PrecBF16::mma(w[b][(3 * ky + kx) * 2 + h], x[kx][h],
                                                                 ky + kx + h == 0 ? cb_f32x4{0.f, 0.f, 0.f, 0.f} : acc[(i - ky) % 3][b]);
                if (i < R + 1) {
                    ad[kx][h] += rowb;
                    x[kx][h] = *reinterpret_cast<const uint4*>(win + ad[kx][h]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        if (i >= 2) emit(i - 2, acc[(i - 2) % 3]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// walk_wgrad for 32 of the input channels (blocks cb, cb + 1, cb even) and 32 of the output channels,
// over one fragment of 32 anchors: acc[tap][ci block][co block], accb[co block].
template <int R>
CB_DEV void walk_wgrad64(const unsigned char* xwin, const unsigned char* dwin, const int (&px)[2], const int (&pd)[2], const int (&c)[2],
                         const int (&skip)[2], uint32_t chx, uint32_t chd, int rowb, cb_f32x4 (&acc)[9][2][2], cb_f32x4 (&accb)[2]) {
    uint32_t ax[2][3], ad[2];
    uint4 x[3][2], d[4][2];
    const uint4 ones = make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
    auto load_d = [&](uint4 (&dst)[2], int i) CB_INLINE_LAMBDA {
        const uint32_t a0 = i >= skip[0] ? ad[0] : 0u, a1 = i >= skip[1] ? ad[1] : 0u;
#pragma unroll
        for (int co = 0; co < 2; ++co) {   // the next channel block's chunk: address bit 5
            const uint2 lo = lds_read_tr16(dwin + (a0 ^ uint32_t(co * 32))), hi = lds_read_tr16(dwin + (a1 ^ uint32_t(co * 32)));
            dst[co] = make_uint4(lo.x, lo.y, hi.x, hi.y);
        }
    };
    auto load_x = [&](int kx, int ci) CB_INLINE_LAMBDA {
        const uint2 lo = lds_read_tr16(xwin + (ax[0][kx] ^ uint32_t(ci * 32))), hi = lds_read_tr16(xwin + (ax[1][kx] ^ uint32_t(ci * 32)));
        x[kx][ci] = make_uint4(lo.x, lo.y, hi.x, hi.y);
    };
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        ad[h] = uint32_t(pd[h]) * 128 + walk64_ch(uint32_t(c[h] + 1), chd);
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) ax[h][kx] = uint32_t(px[h] + kx) * 128 + walk64_ch(uint32_t(c[h] + kx), chx);
    }
    load_d(d[0], 0);
#pragma unroll
    for (int kx = 0; kx < 3; ++kx)
#pragma unroll
        for (int ci = 0; ci < 2; ++ci) load_x(kx, ci);
#pragma unroll
    for (int i = 0; i < R + 2; ++i) {
        if (i + 1 < R) {
            ad[0] += rowb;
            ad[1] += rowb;
            load_d(d[(i + 1) % 4], i + 1);
        }
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) {
#pragma unroll
            for (int ci = 0; ci < 2; ++ci)
#pragma unroll
                for (int ky = 2; ky >= 0; --ky)
                    if (i >= ky && i - ky < R)
#pragma unroll
                        for (int co = 0; co < 2; ++co)
                            acc[3 * ky + kx][ci][co] = PrecBF16::mma(d[(i - ky) % 4][co], x[kx][ci], acc[3 * ky + kx][ci][co]);
            __builtin_amdgcn_sched_barrier(0);
            if (i < R + 1) {
                ax[0][kx] += rowb;
                ax[1][kx] += rowb;
                load_x(kx, 0);
                load_x(kx, 1);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (i < R)
#pragma unroll
            for (int co = 0; co < 2; ++co) accb[co] = PrecBF16::mma(d[i % 4][co], ones, accb[co]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

}  // namespace cb
