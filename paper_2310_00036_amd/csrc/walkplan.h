// Host side of the column-walk kernels: the sizes of their LDS windows and the tile shape of a
// launch (frames and rows per tile, rows per walk), from the problem size and the compute units.
// Plain C++ without HIP, so that the rules can be compiled and checked on any machine.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#ifdef __HIPCC__
#define CB_HD __host__ __device__
#else
#define CB_HD
#endif

namespace cb {

// A window holds F frames of `rows` image rows at a row pitch of W + 1 pixels (column 0 is zero
// padding and serves both sides) and one pixel past the end, in whole blocks of 1 KB, `px` bytes
// per pixel.
CB_HD inline int walk_pitch(int W) { return W + 1; }
CB_HD inline int walk_win_bytes(int px, int F, int rows, int W) {
    return ((F * rows * walk_pitch(W) + 1) * px + 1023) / 1024 * 1024;
}

// Workgroups added to a launch whose own `parts` leave some of its `room` free, to do the pending
// reduces (`blocks` blocks of 64 entries in all, about 2.3 us each; pending_helper in common.h) beside
// its tiles. Without them the tiles wait for ceil(blocks / parts) blocks in turn: 8 frames of 9x9 with
// 32 channels 32 us a launch in a chain against 9, 116 of 21x21 24 against 18; 2 of 11x11 with 64
// channels 132 against 10, 87 of 12x9 28 against 16. None where they would take more than twice as many
// in turn, which shows: 119 of 42x42 with 16 channels, 5 blocks for each of 18 against 1, 23 us against 20.
inline int pend_helpers(int blocks, int parts, int room) {
    const int spare = std::min(room - parts, blocks);
    return spare > 0 && blocks <= 2 * spare * ((blocks + parts - 1) / parts) ? spare : 0;
}

// Rows a wave walks (its filling counted as 0.7 rows per walk) where `waves` waves take groups of
// gw anchors, segments of R <= rows rows; nseg: segments per column.
inline double walk_rows(int rows, int cols, int gw, int waves, int R, int& nseg) {
    nseg = (rows + R - 1) / R;
    return double(((nseg * cols + gw - 1) / gw + waves - 1) / waves) * (R + 0.7);
}

// The tile heights worth trying: every TH that splits H into nb = 1 .. H balanced bands, f(nb, TH).
template <class Fn>
inline void walk_bands(int H, Fn&& f) {
    for (int nb = 1; nb <= H; ++nb) {
        const int TH = (H + nb - 1) / nb;
        if (nb == 1 || (H + TH - 1) / TH == nb) f(nb, TH);
    }
}
constexpr int kWalkMaxF = 16;    // frames per tile
inline int walk_frames(int64_t n, int nb) { return nb > 1 ? 1 : int(std::min<int64_t>(n, kWalkMaxF)); }
inline int walk_tiles(int64_t n, int F, int nb) { return int((n + F - 1) / F) * nb; }

// The cheapest of the shapes that `shapes` offers; false where none fits.
template <class Tile, class Shapes>
inline bool walk_choose(Shapes&& shapes, Tile& t, size_t& lds, double* us = nullptr) {
    double best = 1e30;
    shapes([&](const Tile& c, size_t bytes, double cost) {
        if (cost < best) { best = cost; t = c; lds = bytes; }
    });
    if (us) *us = best;
    return best < 1e30;
}

// ---------------------------------------------------------------- 32-channel block forward
struct RwGeom {
    static constexpr int C = 32, NW = 4, NT = 256, KS = 9, MAXR = 7;   // kernels exist for 1 .. MAXR rows per walk
    static constexpr int MAXS = 11;                  // x-window staging slots per lane
    static constexpr int WFRAG = 2 * KS * 1024;      // one convolution's A fragments (bytes)
    static constexpr size_t LDS_TARGET = 80 * 1024;  // two workgroups per CU
    // frames of which neither a band of one row (wider than 139) nor the whole fits in that: one workgroup
    // per CU, walks of a row or two (the slots' offsets cost every other launch 2%)
    static constexpr int WIDE_MAXS = 21, WIDE_MAXR = 2;
};

struct RwTile {
    int wide;                    // the kernel of wide frames
    int F, TH, nbands, ntiles;   // frames per tile (1 with several bands per frame), rows per band
    int ho;                      // 1: t has a halo row either side (several bands)
    int t_off;                   // LDS bytes of the t window (the x window is at 0)
    int R, nseg1, nseg2;         // rows per walk (the kernel's R), segments of a column: conv1, conv2
    float inv_W, inv_c, inv_TW, inv_xpf;   // 1 / W, 1 / (F * W), 1 / row pitch, 1 / x-window pixels per frame
};

// Every tile shape that fits, f(tile, lds, cost). A tile is F whole frames or a band of one; a wave
// walks ceil(groups / NW) groups of 16 anchors per convolution, R rows each. The cost, in
// microseconds, is rounds of tiles over the resident workgroups (two per CU; a last round with one
// tile per CU at most counts 0.6) times what a tile was measured to take: its rows walked and its
// memory traffic add up, 0.24 us a row, 0.055 a KB and 0.4 for the rest (least squares over every
// shape of 130 problem sizes, 1 .. 8192 frames of 8x12 .. 150x90; the shape chosen takes 1.2% longer
// than the best one on average). With the longer of the two terms instead, all row counts tied
// wherever the traffic was longer, and walks of a single row were taken, which reuse nothing:
// 2048 frames of 21x21 46.8 us against 38.3 with R = 7, 8192 of 21x21 191 against 151, 2048 of 42x42
// 205 against 190, 2048 of 11x11 19.1 against 17.3.
template <class Fn>
inline void rw_shapes(int64_t n, int H, int W, int cus, Fn&& f) {
    using G = RwGeom;
    auto windows = [&](int F, int TH, int ho, int& xb) {
        xb = walk_win_bytes(64, F, TH + 2 + 2 * ho, W);
        return size_t(xb) + std::max(walk_win_bytes(64, F, TH + 2, W), 2 * G::WFRAG);
    };
    auto fits = [&](int F, int TH, int ho, bool wide) {
        int xb = 0;
        return windows(F, TH, ho, xb) <= (wide ? 2 : 1) * G::LDS_TARGET && xb <= (wide ? G::WIDE_MAXS : G::MAXS) * G::NW * 1024;
    };
    const bool wide = !fits(1, 1, 1, false) && !fits(1, H, 0, false);
    walk_bands(H, [&](int nb, int TH) {
        const int ho = nb > 1;
        for (int F = 1; F <= walk_frames(n, nb); ++F) {
            if (!fits(F, TH, ho, wide)) break;
            int xb = 0;
            const size_t lds = windows(F, TH, ho, xb);
            RwTile c{};
            c.wide = wide; c.F = F; c.TH = TH; c.ho = ho; c.nbands = nb; c.ntiles = walk_tiles(n, F, nb); c.t_off = xb;
            c.inv_W = 1.f / float(W); c.inv_c = 1.f / float(F * W);
            c.inv_TW = 1.f / float(walk_pitch(W)); c.inv_xpf = 1.f / float((TH + 2 + 2 * ho) * walk_pitch(W));
            const double traffic = double(F) * W * 64 * (3 * TH + 4 * ho) / 1000;
            const int full = c.ntiles / (2 * cus), rest = c.ntiles - full * 2 * cus;
            const double rounds = full + (rest > cus ? 1.0 : rest > 0 ? 0.6 : 0.0);
            for (c.R = 1; c.R <= std::min(TH, wide ? G::WIDE_MAXR : G::MAXR); ++c.R) {
                const double rows = walk_rows(TH + 2 * ho, F * W, 16, G::NW, c.R, c.nseg1) + walk_rows(TH, F * W, 16, G::NW, c.R, c.nseg2);
                f(c, lds, rounds * (0.244 * rows + 0.0546 * traffic + 0.37));
            }
        }
    });
}

// ---------------------------------------------------------------- block backward, 32 and 16 channels
struct RbwGeom {
    static constexpr int C = 32, NW = 8, NT = 512, NS = 4, PX = 64, MAXR = 7;   // NS: waves per role; PX: bytes per pixel
    static constexpr int NBB = 19, PSTRIDE = 2 * NBB * 256;  // partial: [co block][tap x ci block, bias][co][ci]
    static constexpr int MAXD = 6, MAXX = 6, MAXK = 5;       // staging slots per lane: dy; t / x; skip term
    static constexpr int WFRAG = 2 * 9 * 1024;               // one convolution's A fragments (bytes)
    static constexpr int MIN_TAIL = 2 * WFRAG;               // the dt window's memory holds the weights at first
    static constexpr size_t MIN_LDS = 0;
    static constexpr int GW = 64, WW = 1;                    // anchors per weight-gradient group, waves sharing the groups
    // microseconds: a launch; a MB of partial sums; a row walked by a convolution's and by a weight
    // gradient's wave; a KB of a tile's traffic; a tile
    static constexpr double US = 9.3, US_PARTIAL = 0.368, US_CONV = 0.060, US_WGRAD = 0.285, US_KB = 0.0183, US_TILE = 0.68;
};
struct Rbw16Geom {
    static constexpr int C = 16, NW = 8, NT = 512, NS = 4, PX = 32, MAXR = 8;
    static constexpr int NBB = 10, PSTRIDE = NBB * 256;      // partial: [tap, bias][co][ci]
    static constexpr int MAXD = 6, MAXX = 6, MAXK = 5;
    static constexpr int MIN_TAIL = 0;
    static constexpr size_t MIN_LDS = 4 * 20 * 1024;         // the four waves' sums, at the end
    static constexpr int GW = 32, WW = 4;
    static constexpr double US = 9.4, US_PARTIAL = 0.653, US_CONV = 0.104, US_WGRAD = 0.0245, US_KB = 0.0199, US_TILE = 0.81;
};

struct RbwTile {
    int F, TH, nbands, ntiles;
    int ho;                      // 1: dt has a halo row either side (several bands)
    int t_off, x_off, dt_off, sk_off, dt_bytes;   // LDS bytes (the dy window is at 0)
    int R, nsegt, nsegx, nsegw;  // rows per walk (the kernel's R), segments of a column: dt, dx, weight gradients
    int pset;                    // floats per partial set (one per convolution)
    float inv_W, inv_c, inv_TW, inv_dpf, inv_xpf;    // 1 / W, F * W, row pitch, window pixels per frame (dy; t, x, dt)
};

// Every tile shape that fits, f(tile, lds, cost). The cost is the launch with its reduce in
// microseconds, fitted like the forward's over 130 problem sizes for 32 channels and 260 for 16 (the
// estimates of the shapes chosen are within 6% and 4%, the shapes chosen within 1% of the best on
// average). Counting the longer of work and traffic in each phase, and no partial sums, cut launches of
// few frames into one-row bands: 40 frames of 21x21 with 32 channels 23 against 18 us, 128 of 11x11 24
// against 18; and took too tall bands for many: 2048 of 84x84 with 16 channels 658 against 617.
template <class G, class Fn>
inline void rbw_shapes(int64_t n, int H, int W, int cus, size_t limit, Fn&& f) {
    walk_bands(H, [&](int nb, int TH) {
        const int ho = nb > 1;
        for (int F = 1; F <= walk_frames(n, nb); ++F) {
            const int db = walk_win_bytes(G::PX, F, TH + 2 + 2 * ho, W), xb = walk_win_bytes(G::PX, F, TH + 2, W);
            const int kb = (F * TH * W * G::PX + 1023) / 1024 * 1024;
            const size_t lds = size_t(db) + 2 * xb + std::max(xb + kb, G::MIN_TAIL);   // dy; t, x; dt, skip term
            if (lds > limit || kb > G::MAXK * G::NW * 1024 || db > G::MAXD * G::NW * 1024 || xb > G::MAXX * G::NW * 1024) break;
            RbwTile c{};
            c.F = F; c.TH = TH; c.ho = ho; c.nbands = nb; c.ntiles = walk_tiles(n, F, nb);
            c.t_off = db; c.x_off = db + xb; c.dt_off = db + 2 * xb; c.sk_off = c.dt_off + xb; c.dt_bytes = xb;
            c.pset = std::min(cus, c.ntiles) * G::PSTRIDE;
            c.inv_W = 1.f / float(W); c.inv_c = 1.f / float(F * W); c.inv_TW = 1.f / float(walk_pitch(W));
            c.inv_dpf = 1.f / float((TH + 2 + 2 * ho) * walk_pitch(W)); c.inv_xpf = 1.f / float((TH + 2) * walk_pitch(W));
            const double traffic = double(F) * W * G::PX * (5 * TH + 8 * ho) / 1000, partials = 2.0 * c.pset * 4 / 1e6;
            const double rounds = (c.ntiles + cus - 1) / cus;
            for (c.R = 1; c.R <= std::min(TH, G::MAXR); ++c.R) {
                const double conv = walk_rows(TH + 2 * ho, F * W, 16, G::NS, c.R, c.nsegt) + walk_rows(TH, F * W, 16, G::NS, c.R, c.nsegx);
                const double wgrad = 2 * walk_rows(TH, F * W, G::GW, G::WW, c.R, c.nsegw);
                f(c, std::max(lds, G::MIN_LDS),
                  G::US + G::US_PARTIAL * partials + rounds * (G::US_CONV * conv + G::US_WGRAD * wgrad + G::US_KB * traffic + G::US_TILE));
            }
        }
    });
}

// ---------------------------------------------------------------- 16-channel block backward, tile by tile
struct RbtGeom {
    static constexpr int C = 16, NW = 8, NT = 512, PX = 32, NBB = Rbw16Geom::NBB, PSTRIDE = Rbw16Geom::PSTRIDE;
    static constexpr int MAXS = 4;                           // staging slots per lane and window
    static constexpr size_t LDS_TARGET = 80 * 1024;          // two workgroups per CU
    static constexpr size_t MIN_LDS = NW * 4 * 17 * 16;      // earlier launches' reduces
};
struct RbtTile {
    int TH, nbands, ntiles;
    int dy_off, t_off, x_off, dt_off;   // LDS byte offsets; 64 zero bytes at offset 0
    int tx_guard;                       // t / x windows: byte offset of the rear guard pixel
    int dt_bytes;
    int pset;                           // floats per partial set (the launcher's, from its grid)
    float inv_W, inv_TW;
};

// The balanced bands of the fewest tiles that fit; false where none does (frames wider than 202). us:
// the estimated time with its reduce, like the walks' (fitted over 170 problem sizes; two workgroups
// per CU, a last round of one per CU counts 0.6).
inline bool rbt_shape(int64_t n, int H, int W, int cus, size_t limit, RbtTile& t, size_t& lds, double& us) {
    using G = RbtGeom;
    const int TW = W + 2;
    auto layout = [&](int th) {
        const int dyb = ((th + 4) * TW * 2 + 63) / 64 * 1024;
        const int txb = ((th + 2) * TW * 2 + 63) / 64 * 1024 + 2 * G::PX;   // + a guard pixel either side
        t.dt_bytes = (th + 2) * TW * G::PX;
        t.dy_off = 64; t.t_off = t.dy_off + dyb; t.x_off = t.t_off + txb; t.dt_off = t.x_off + txb;
        t.tx_guard = txb - 2 * G::PX;
        return size_t(t.dt_off) + t.dt_bytes;
    };
    auto fits = [&](int th) { return (th + 4) * TW * 2 <= G::MAXS * G::NT; };
    int th = H;
    while (th > 1 && (layout(th) > G::LDS_TARGET || !fits(th))) --th;
    if (layout(th) > limit || !fits(th)) return false;
    const int nb0 = (H + th - 1) / th;
    t.TH = (H + nb0 - 1) / nb0;
    t.nbands = (H + t.TH - 1) / t.TH;
    t.ntiles = walk_tiles(n, 1, t.nbands);
    t.inv_W = 1.f / float(W);
    t.inv_TW = 1.f / float(TW);
    lds = std::max(layout(t.TH), G::MIN_LDS);
    const int full = t.ntiles / (2 * cus), rest = t.ntiles - full * 2 * cus;
    const double rounds = full + (rest > cus ? 1.0 : rest > 0 ? 0.6 : 0.0);
    auto groups = [&](int rows) { return ((rows * W + 15) / 16 + G::NW - 1) / G::NW; };
    const double partials = 2.0 * std::min(2 * cus, t.ntiles) * G::PSTRIDE * 4 / 1e6;
    const double wgrad = t.TH * TW / 32.0, traffic = double(W) * G::PX * (5 * t.TH + 8) / 1000;
    us = 11.9 + 0.956 * partials + rounds * (0.112 * (groups(t.TH + 2) + groups(t.TH)) + 0.268 * wgrad + 0.0264 * traffic + 0.94);
    return true;
}

// The 16-channel block backward's launch: whichever form's estimate is the shorter.
struct Rb16Plan {
    bool tiles;      // tile by tile (u), else column walks (t)
    RbwTile t;
    RbtTile u;
};
inline bool rb16_choose(int64_t n, int H, int W, int cus, size_t limit, Rb16Plan& p, size_t& lds) {
    size_t walk_lds = 0, tile_lds = 0;
    double walk_us = 0, tile_us = 0;
    const bool walk = walk_choose([&](auto&& f) { rbw_shapes<Rbw16Geom>(n, H, W, cus, limit, f); }, p.t, walk_lds, &walk_us);
    const bool tile = rbt_shape(n, H, W, cus, limit, p.u, tile_lds, tile_us);
    p.tiles = tile && (!walk || tile_us < walk_us);
    lds = p.tiles ? tile_lds : walk_lds;
    return walk || tile;
}

// ---------------------------------------------------------------- 64-channel conv backward
struct Cw64Geom {
    static constexpr int C = 64, NW = 8, NT = 512, NS = 4, MAXR = 7;   // NS: waves per role
    static constexpr int NBB = 37, PSTRIDE = 4 * NBB * 256;  // partial: [co block][tap x ci block, bias][co][ci]
    static constexpr int MAXS = 10;                          // staging slots per lane and window
    static constexpr size_t WBYTES = 72 * 1024;              // the weights' A fragments, before the windows
};
struct Cw64Tile {
    int F, TH, nbands, ntiles;
    int ho;                    // several bands per frame
    int win;                   // window bytes; LDS: dy, x of buffer 0, then of buffer 1
    int R, nsegd, nsegw;       // rows per walk (the kernel's R), segments of a column: dx, weight gradients
    int parts;                 // workgroups
    float inv_W, inv_c, inv_TW, inv_pf;   // 1 / W, F * W, row pitch, window pixels per frame
};

// Every tile shape that fits, f(tile, lds, cost). The cost in microseconds, fitted like the forward's
// over 90 problem sizes: each workgroup leaves 152 KB of partial sums to be added (0.29 us a MB), a
// tile takes 0.55 us per row walked and 0.019 per KB of traffic. Without the partials' term, launches
// of few frames were split into one- and two-row bands over all CUs: 40 frames of 11x11 28.9 us in 240
// workgroups, 18.6 in 40; 8 of 24x24 27.9 against 19.2.
template <class Fn>
inline void cw64_shapes(int64_t n, int H, int W, int cus, size_t limit, Fn&& f) {
    using G = Cw64Geom;
    walk_bands(H, [&](int nb, int TH) {
        const int ho = nb > 1;
        for (int F = 1; F <= walk_frames(n, nb); ++F) {
            Cw64Tile c{};
            c.win = walk_win_bytes(128, F, TH + 2, W);
            if (4 * size_t(c.win) > limit || c.win > G::MAXS * G::NS * 1024) break;
            c.F = F; c.TH = TH; c.ho = ho; c.nbands = nb; c.ntiles = walk_tiles(n, F, nb);
            c.parts = std::min(cus, c.ntiles);
            c.inv_W = 1.f / float(W); c.inv_c = 1.f / float(F * W); c.inv_TW = 1.f / float(walk_pitch(W));
            c.inv_pf = 1.f / float((TH + 2) * walk_pitch(W));
            const double traffic = double(F) * W * 128 * (4 * TH + 4 * ho) / 1000, partials = double(c.parts) * G::PSTRIDE * 4 / 1e6;
            const double rounds = (c.ntiles + cus - 1) / cus;
            for (c.R = 1; c.R <= std::min(TH, G::MAXR); ++c.R) {
                const double rows = walk_rows(TH, F * W, 16, 2, c.R, c.nsegd);
                walk_rows(TH, F * W, 32, 1, c.R, c.nsegw);   // (in step with dx's: one wave, twice the anchors)
                f(c, std::max(4 * size_t(c.win), G::WBYTES), 0.294 * partials + rounds * (0.550 * rows + 0.0185 * traffic + 0.11));
            }
        }
    });
}

}  // namespace cb
