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
    // One level per lane, where packed strips make up for the narrow loads, or
    // more where a column fills them.  FP32: fitted to 18 grids with and without
    // the epilogue, 4 % slower than the best shape; FP64: 8 grids, 3 %.  FP32
    // above 12 M points of up to 64 levels: four-row strips in workgroups of
    // four, which read fewer rows twice; there is little between them at the
    // line (430x430x64, 11.8 M points: 63.7 us against 68.2, with the epilogue
    // 87.8 against 87.4), and 81 against 97 us at 512x512x64.
    const auto pick = [&](const ShapeCost *s, int n) { return cheapest_shape(s, n, a.nz, a.ny, a.nx, true); };
    static const ShapeCost tall[] = {{1, 4, 4, 2, 0, 64, 1024, 1.75}};
    if (dt == PW_F64) {
        static const ShapeCost s[] = {{1, 2, 1, 1, 0, 64, 1024, 1.00}, {2, 2, 1, 1, 0, 128, 1024, 1.23}};
        return pick(s, 2);
    }
    if (dt == PW_F32 && a.nz <= 64 && a.nx * a.ny * a.nz >= 12000000) return pick(tall, 1);
    if (dt == PW_F32) {
        static const ShapeCost s[] = {{1, 1, 1, 1, 0, 64, 2048, 1.00}, {1, 2, 1, 1, 0, 64, 2048, 1.875},
                                      {2, 4, 1, 1, 0, 128, 1024, 2.70}, {4, 2, 1, 1, 0, 256, 1024, 2.00}};
        return pick(s, 4);
    }
    // 16-bit storage: 170 grids, 7 % slower than the best shape.  With the shapes
    // given by the number of levels and one-level lanes counted as plain strips
    // 24 %: BF16 308x56x68 17.6 -> 10.6 us, 545x313x70 117 -> 70.
    static const ShapeCost s[] = {{1, 1, 1, 1, 0, 64, 2048, 1.00, 0.3}, {1, 2, 1, 1, 0, 64, 2048, 1.32, 1.9},
                                  {1, 4, 1, 1, 0, 64, 2048, 2.81, 1.2}, {2, 2, 1, 1, 0, 128, 2048, 1.99, 3.7},
                                  {4, 2, 1, 1, 0, 256, 2048, 2.73, 5.0}};
    return pick(s, 5);
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
