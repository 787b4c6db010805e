// The tile shapes that walkplan.h chooses, for tests/test_walk_plans.py (plain C++, no GPU).
#include "../paper_2310_00036_amd/csrc/walkplan.h"

using namespace cb;

constexpr size_t kLds = 160 * 1024;   // of a CU

// out: F, TH, bands, tiles, R, LDS bytes; 0 where no shape fits.
template <class Tile, class Shapes>
static int choose(Shapes&& shapes, int64_t* out) {
    Tile t{};
    size_t lds = 0;
    if (!walk_choose(shapes, t, lds)) return 0;
    const int64_t v[6] = {t.F, t.TH, t.nbands, t.ntiles, t.R, int64_t(lds)};
    std::copy(v, v + 6, out);
    return 1;
}

extern "C" int walk_plan(const char* kind, int64_t n, int H, int W, int cus, int64_t* out) {
    switch (kind[0] * 256 + kind[1]) {
        case 'f' * 256 + '3': return choose<RwTile>([&](auto&& f) { rw_shapes(n, H, W, cus, f); }, out);
        case 'b' * 256 + '3': return choose<RbwTile>([&](auto&& f) { rbw_shapes<RbwGeom>(n, H, W, cus, kLds, f); }, out);
        case 'b' * 256 + '1': return choose<RbwTile>([&](auto&& f) { rbw_shapes<Rbw16Geom>(n, H, W, cus, kLds, f); }, out);
        case 't' * 256 + '1': {   // the 16-channel block backward's launch; R = 0: tile by tile
            Rb16Plan p{};
            size_t lds = 0;
            if (!rb16_choose(n, H, W, cus, kLds, p, lds)) return 0;
            const int64_t u[6] = {1, p.u.TH, p.u.nbands, p.u.ntiles, 0, int64_t(lds)}, w[6] = {p.t.F, p.t.TH, p.t.nbands, p.t.ntiles, p.t.R, int64_t(lds)};
            std::copy(p.tiles ? u : w, (p.tiles ? u : w) + 6, out);
            return 1;
        }
        case 'c' * 256 + '6': return choose<Cw64Tile>([&](auto&& f) { cw64_shapes(n, H, W, cus, kLds, f); }, out);
    }
    return 0;
}

extern "C" int walk_pend_helpers(int blocks, int parts, int room) { return pend_helpers(blocks, parts, room); }
