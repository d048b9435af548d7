// z-fastest forward: launch-shape rules, default shape and dispatch to the
// per-storage-type translation units (the kernel is in pw_zfast_impl.h).
#include "pw_internal.h"

namespace pw {

bool zfast_tile_supported(const TileCfg &c, pw_dtype dt) {
    if (c.zlen < 1 || c.wpb < 1 || c.wpb > 8 || (c.depth != 1 && c.depth != 2) || c.share != 0) return false;
    const bool pz_ok = c.px == 1 || c.px == 2 || (c.px == 4 && dt != PW_F64);
    const bool ry_ok = c.ry == 1 || c.ry == 2 || (c.ry == 4 && c.px <= 2) || (c.ry == 8 && c.px == 1);
    return pz_ok && ry_ok;
}

TileCfg default_zfast_tile(const FwdArgs &a, pw_dtype dt) {
    // One level per lane where packed strips make up for the narrow loads, more
    // where a column fills them.  FP32: fitted to 18 grids with and without the
    // epilogue, 4 % slower than the best shape; FP64: 8 grids, 3 %.  Above 12 M
    // points of up to 64 levels four-row strips in workgroups of four, which
    // read fewer rows twice: 512x512x64 108 us against 117 (accumulate, FP32).
    static const ShapeCost tall[] = {{1, 4, 4, 2, 0, 64, 1024, 1.75, true}};
    if (dt == PW_F64) {
        static const ShapeCost s[] = {{1, 2, 1, 1, 0, 64, 1024, 1.00, true}, {2, 2, 1, 1, 0, 128, 1024, 1.23}};
        return cheapest_shape(s, 2, a.nz, a.ny, a.nx);
    }
    if (a.nz <= 64 && a.nx * a.ny * a.nz >= 12000000) return cheapest_shape(tall, 1, a.nz, a.ny, a.nx);
    if (dt == PW_F32) {
        static const ShapeCost s[] = {{1, 1, 1, 1, 0, 64, 2048, 1.00, true}, {1, 2, 1, 1, 0, 64, 2048, 1.875, true},
                                      {2, 4, 1, 1, 0, 128, 1024, 2.70}, {4, 2, 1, 1, 0, 256, 1024, 2.00}};
        return cheapest_shape(s, 4, a.nz, a.ny, a.nx);
    }
    // 16-bit storage: as many levels per lane as a column fills
    static const ShapeCost s[] = {{1, 2, 1, 1, 0, 64, 2048, 0.96}, {2, 2, 1, 1, 0, 128, 1024, 0.90},
                                  {4, 2, 1, 1, 0, 256, 1024, 1.05}};
    return cheapest_shape(s, a.nz > 128 ? 3 : a.nz > 64 ? 2 : 1, a.nz, a.ny, a.nx);
}

pw_status launch_zfast(const FwdArgs &a, pw_dtype dt, const TileCfg &cfg, hipStream_t s) {
    if (!zfast_tile_supported(cfg, dt)) return fail(PW_ERR_INVALID_ARG, "unsupported z-fastest tile configuration");
    if (a.epilogue && a.nz < cfg.px) {
        // columns shorter than one lane's levels: one-level lanes (the same
        // bits), see load_zepi
        TileCfg c = cfg;
        c.px = 1;
        return launch_zfast(a, dt, c, s);
    }
    switch (dt) {
        case PW_F32: return launch_zfast_f32(a, cfg, s);
        case PW_F64: return launch_zfast_f64(a, cfg, s);
        case PW_BF16: return launch_zfast_bf16(a, cfg, s);
        case PW_F16: return launch_zfast_f16(a, cfg, s);
    }
    return fail(PW_ERR_UNSUPPORTED, "dtype %d", static_cast<int>(dt));
}

}  // namespace pw
