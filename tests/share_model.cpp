// CPU model of a launch's tile shares: the library's own host and device functions, called for every workgroup.
#include "../paper_2603_01399_amd/csrc/shares.hpp"

using namespace quasar;

struct Params {
    int T, tq, tr, groups, xcd_shift;
};

template <int TU, bool DEAL, bool EVEN>
static int walk(const Params &p, int b, int *tiles) {
    const TileShare<TU, DEAL, EVEN> share(p, b);
    for (int tl = 0; tl < TU * share.units; ++tl) tiles[tl] = share.tile(tl);
    return TU * share.units;
}

// Tiles of workgroup b of a slice, in its order (form: 0 dealt, 1 contiguous, 2 contiguous as tile_split cuts); returns how many.
extern "C" int share_model(int T, int groups, int ksplit, int unit, int form, int b, int *tiles) {
    Params p{T};
    share_tiles(p, groups, ksplit, unit);
    if (unit == 2) return form == 0 ? walk<2, true, false>(p, b, tiles) : (form == 1 ? walk<2, false, false>(p, b, tiles) : walk<2, false, true>(p, b, tiles));
    return form == 0 ? walk<1, true, false>(p, b, tiles) : (form == 1 ? walk<1, false, false>(p, b, tiles) : walk<1, false, true>(p, b, tiles));
}
