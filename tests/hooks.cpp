// Host functions of the library that its interface does not show, for tests
// (built by hooks.py against the built library).
#include <vector>

#include "pw_internal.h"

// The strip count that the launch rule and the launches share.
extern "C" int64_t count_strips(int64_t lead, int64_t rows, int cols, int ry, int may_pack, int *packed) {
    const pw::Strips s = pw::strips_of(lead, rows, cols, ry, may_pack != 0);
    *packed = s.packed;
    return s.count;
}

// The rule over one shape of strips ry rows high.
extern "C" int march_length(int64_t lead, int64_t rows, int64_t march, int cols, int ry, int slots, double start,
                            int may_pack) {
    const pw::ShapeCost s{cols / 64, ry, 1, 1, 0, cols, slots, 1.0, start};
    return pw::cheapest_shape(&s, 1, lead, rows, march, may_pack != 0).zlen;
}

// The default forward (zfast 0) or z-fastest shape of a grid, without boundary
// rules (0), with remapped reads (1) or with value rules too (2).
extern "C" void pick(int zfast, int dtype, int64_t nx, int64_t ny, int64_t nz, int rules, int32_t out[6]) {
    pw::FwdArgs a{};
    a.nx = nx;
    a.ny = ny;
    a.nz = nz;
    a.h = 1;
    if (rules) a.bcx = a.bcy = PW_HALO_PERIODIC;
    if (rules > 1) a.bcv = 2u;
    const pw_dtype dt = static_cast<pw_dtype>(dtype);
    const pw::TileCfg c = zfast ? pw::default_zfast_tile(a, dt) : pw::default_forward_tile(a, dt);
    const int v[6] = {c.px, c.ry, c.zlen, c.wpb, c.depth, c.share};
    for (int i = 0; i < 6; ++i) out[i] = v[i];
}

// The shapes that tuning a batch times, the batch's own first.
namespace pw {
std::vector<TileCfg> batch_candidates(const TileCfg &start);
}
extern "C" int batch_candidates(const int32_t start[6], int32_t (*out)[6], int most) {
    int n = 0;
    for (const pw::TileCfg &c : pw::batch_candidates({start[0], start[1], start[2], start[3], start[4], start[5]})) {
        if (n == most) break;
        const int32_t v[6] = {c.px, c.ry, c.zlen, c.wpb, c.depth, c.share};
        for (int i = 0; i < 6; ++i) out[n][i] = v[i];
        ++n;
    }
    return n;
}
