// Autotuner for single-grid launches and its process-wide cache.
//
// The launch shape (columns per lane, rows per strip, z-chunks, wavefronts
// per workgroup) changes only speed, never results.  pw_tune times candidate
// shapes on scratch grids and keeps the fastest per kernel kind, dtype and
// shape class (the power-of-two ceilings of nx, ny, nz); pw_advect and
// pw_advect_adjoint use it when called without a tile.  The vertical cut is
// stored as a number of z-chunks, so one entry serves every nz of its class.
// With PWADV_TUNE_CACHE set, the table is read from that file on first use
// and rewritten after every pw_tune (one entry per line, plain text).
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <tuple>
#include <vector>

#include "pw_internal.h"

namespace pw {
namespace {

int ceil_log2(int64_t x) {
    int l = 0;
    while ((int64_t(1) << l) < x) ++l;
    return l;
}

using Key = std::tuple<int, int, int, int, int>;   // kind, dtype, log2 nx, ny, nz
struct Entry {
    int px, ry, nzc, wpb, depth, share;
    bool measured;   // from pw_tune or the cache file (saved); false for built-in entries
};

std::mutex g_mu;
std::map<Key, Entry> g_table;
bool g_loaded = false;

Key make_key(TuneKind kind, const pw_grid *g, pw_dtype dt) {
    return Key(static_cast<int>(kind), static_cast<int>(dt), ceil_log2(g->nx), ceil_log2(g->ny), ceil_log2(g->nz));
}

const char *cache_path() {
    const char *p = std::getenv("PWADV_TUNE_CACHE");
    return (p && *p) ? p : nullptr;
}

// Shapes chosen by pw_tune on an MI355X for the shape classes the library is
// benchmarked on (generated by paper_2301_13016_amd/tune_defaults.py); used
// when neither this process nor the cache file has a better entry.
struct BuiltinEntry {
    int kind, dt, lx, ly, lz, px, ry, nzc, wpb, depth, share;   // rows without share: 0
};
const BuiltinEntry kBuiltin[] = {
#include "pw_tune_defaults.inc"
};

// Called with g_mu held.
void load_locked() {
    if (g_loaded) return;
    g_loaded = true;
    for (const BuiltinEntry &e : kBuiltin)
        if (e.px > 0)
            g_table[Key(e.kind, e.dt, e.lx, e.ly, e.lz)] = Entry{e.px, e.ry, e.nzc, e.wpb, e.depth, e.share, false};
    const char *path = cache_path();
    if (!path) return;
    FILE *f = std::fopen(path, "r");
    if (!f) return;   // a missing cache is an empty one
    char line[256];
    while (std::fgets(line, sizeof line, f)) {
        // "pwadv-tune-v3 kind dtype lx ly lz px ry nzc wpb depth share"; v2 lines have no share (0),
        // v1 lines neither depth (1)
        int kind, dt, lx, ly, lz, px, ry, nzc, wpb, depth = 1, share = 0;
        const bool v3 = std::sscanf(line, "pwadv-tune-v3 %d %d %d %d %d %d %d %d %d %d %d", &kind, &dt, &lx, &ly,
                                    &lz, &px, &ry, &nzc, &wpb, &depth, &share) == 11;
        const bool v2 = !v3 && std::sscanf(line, "pwadv-tune-v2 %d %d %d %d %d %d %d %d %d %d", &kind, &dt, &lx, &ly,
                                           &lz, &px, &ry, &nzc, &wpb, &depth) == 10;
        const bool v1 = !v3 && !v2 && std::sscanf(line, "pwadv-tune-v1 %d %d %d %d %d %d %d %d %d", &kind, &dt, &lx,
                                                  &ly, &lz, &px, &ry, &nzc, &wpb) == 9;
        if ((v1 || v2 || v3) && nzc >= 1 && wpb >= 1 && wpb <= 8 && px >= 1 && ry >= 1 &&
            (depth == 1 || depth == 2) && share >= 0 && share <= 2)
            g_table[Key(kind, dt, lx, ly, lz)] = Entry{px, ry, nzc, wpb, depth, share, true};
        // anything else (corrupt or foreign lines) is ignored
    }
    std::fclose(f);
}

void save_locked() {
    const char *path = cache_path();
    if (!path) return;
    const std::string tmp = std::string(path) + ".tmp";
    FILE *f = std::fopen(tmp.c_str(), "w");
    if (!f) return;
    for (const auto &kv : g_table) {
        if (!kv.second.measured) continue;
        int kind, dt, lx, ly, lz;
        std::tie(kind, dt, lx, ly, lz) = kv.first;
        std::fprintf(f, "pwadv-tune-v3 %d %d %d %d %d %d %d %d %d %d %d\n", kind, dt, lx, ly, lz, kv.second.px,
                     kv.second.ry, kv.second.nzc, kv.second.wpb, kv.second.depth, kv.second.share);
    }
    std::fclose(f);
    std::rename(tmp.c_str(), path);
}

TileCfg entry_to_cfg(const Entry &e, int64_t zextent) {
    TileCfg c;
    c.px = e.px;
    c.ry = e.ry;
    c.wpb = e.wpb;
    c.depth = e.depth;
    c.share = e.share;
    c.zlen = static_cast<int>((zextent + e.nzc - 1) / e.nzc);
    if (c.zlen < 1) c.zlen = 1;
    return c;
}

// Timing helper: mean milliseconds of `reps` launches, as a graph that is
// replayed once before; launch(i) runs on buffer set i (the caller rotates its
// sets, so that repeats do not come out of the 256 MB MALL).  Launched one by
// one, kernels shorter than the host's time per launch all look alike: at
// 32x32x64 that kept a shape of 4.2 us where the untuned one takes 2.5.
template <typename F> float time_ms(F launch, hipStream_t s, int reps, pw_status *st) {
    hipEvent_t a, b;
    if (hipEventCreate(&a) != hipSuccess) return -1.f;
    if (hipEventCreate(&b) != hipSuccess) {
        (void)hipEventDestroy(a);
        return -1.f;
    }
    float ms = -1.f;
    hipGraph_t g = nullptr;
    hipGraphExec_t x = nullptr;
    *st = PW_OK;
    if (hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal) == hipSuccess) {
        for (int i = 0; i < reps && *st == PW_OK; ++i) *st = launch(i);
        const hipError_t e = hipStreamEndCapture(s, &g);
        if (*st == PW_OK && e == hipSuccess && hipGraphInstantiate(&x, g, nullptr, nullptr, 0) == hipSuccess &&
            hipGraphLaunch(x, s) == hipSuccess && hipEventRecord(a, s) == hipSuccess &&
            hipGraphLaunch(x, s) == hipSuccess && hipEventRecord(b, s) == hipSuccess &&
            hipEventSynchronize(b) == hipSuccess && hipEventElapsedTime(&ms, a, b) == hipSuccess)
            ms /= reps;
        else
            ms = -1.f;
    }
    if (x) (void)hipGraphExecDestroy(x);
    if (g) (void)hipGraphDestroy(g);
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    return ms;
}

// Two-stage selection after a warm-up (the clocks settle over the first
// hundred or so launches): every candidate timed over 12 launches, then the
// eight fastest re-timed in three interleaved rounds of 40 launches each
// (forward, backward, forward order), ranked by the median of their rounds.
// Interleaving spreads slow drifts of the clock over all finalists, and the
// median drops a round that one disturbance slowed.  (A single pass of 30
// launches over five finalists had ranked shapes 1.8 % and 3.7 % apart the
// wrong way round.)  *best is the shape that untuned calls take, a candidate
// like the others: tuning must not leave a grid slower (32x32x64, whose march
// the rule cuts into single levels, shorter than any candidate below).
template <typename F>
pw_status pick_fastest(std::vector<TileCfg> cands, F launch, hipStream_t s, TileCfg *best) {
    cands.insert(cands.begin(), *best);
    std::vector<std::pair<float, size_t>> t;
    if (!cands.empty()) {
        pw_status ls = PW_OK;
        (void)time_ms([&](int rep) { return launch(cands[0], rep); }, s, 100, &ls);
        if (ls != PW_OK) return ls;
    }
    for (size_t i = 0; i < cands.size(); ++i) {
        pw_status ls = PW_OK;
        const float ms = time_ms([&](int rep) { return launch(cands[i], rep); }, s, 12, &ls);
        if (ls != PW_OK) return ls;
        if (ms > 0.f) t.emplace_back(ms, i);
    }
    if (t.empty()) return PW_OK;   // keep the caller's default
    std::sort(t.begin(), t.end());
    const size_t nf = std::min<size_t>(t.size(), 8);
    constexpr int kRounds = 3;
    std::vector<std::vector<float>> rounds(nf);
    for (int r = 0; r < kRounds; ++r) {
        for (size_t q = 0; q < nf; ++q) {
            const size_t f = (r % 2 == 0) ? q : nf - 1 - q;
            pw_status ls = PW_OK;
            const float ms = time_ms([&](int rep) { return launch(cands[t[f].second], rep); }, s, 40, &ls);
            if (ls != PW_OK) return ls;
            rounds[f].push_back(ms);
        }
    }
    float best_ms = -1.f;
    for (size_t f = 0; f < nf; ++f) {
        std::vector<float> &v = rounds[f];
        if (std::any_of(v.begin(), v.end(), [](float x) { return x <= 0.f; })) continue;
        std::sort(v.begin(), v.end());
        const float med = v[v.size() / 2];
        if (best_ms < 0.f || med < best_ms) {
            best_ms = med;
            *best = cands[t[f].second];
        }
    }
    return PW_OK;
}

struct DevBuf {
    void *p = nullptr;
    ~DevBuf() {
        if (p) (void)hipFree(p);
    }
    hipError_t alloc(size_t n) { return hipMalloc(&p, n); }
};

}  // namespace

// Extent of the marched axis, which the stored chunk count divides: z for the
// x-fastest kernels (padded for the adjoint), x for the z-fastest one.
static int64_t march_extent(TuneKind kind, const pw_grid *grid) {
    switch (kind) {
        case TuneKind::Adjoint: return grid->nz + 2 * grid->halo;
        case TuneKind::Zfast: return grid->nx;
        default: return grid->nz;
    }
}

int env_forward_tile(pw_tile *t) {
    const char *e = std::getenv("PWADV_TILE");
    if (!e || !*e) return 0;
    long v[6] = {0, 0, 0, 4, 1, 0};
    int n = 0;
    const char *p = e;
    while (n < 6) {
        char *end = nullptr;
        const long x = std::strtol(p, &end, 10);
        if (end == p || x < -(1L << 30) || x > (1L << 30)) return -1;
        v[n++] = x;
        p = end;
        if (*p != 'x' && *p != ',') break;
        ++p;
    }
    if (*p != '\0' || n < 3) return -1;
    *t = pw_tile{static_cast<int32_t>(v[0]), static_cast<int32_t>(v[1]), static_cast<int32_t>(v[2]),
                 static_cast<int32_t>(v[3]), static_cast<int32_t>(v[4]), static_cast<int32_t>(v[5])};
    return 1;
}

bool lookup_tuned(TuneKind kind, const pw_grid *grid, pw_dtype dt, TileCfg *cfg) {
    std::lock_guard<std::mutex> lk(g_mu);
    load_locked();
    auto it = g_table.find(make_key(kind, grid, dt));
    if (it == g_table.end()) return false;
    // A built-in entry holds for the power-of-two grid it was measured on (aligned rows, whole strips); other
    // sizes of its class are better served by the cost rule: 201x143x117 FP32 29 us with the entry of
    // 256x256x128, 19 us with the rule's shape.
    auto power = [](int64_t n) { return (n & (n - 1)) == 0; };
    if (!it->second.measured && !(power(grid->nx) && power(grid->ny) && power(grid->nz))) return false;
    *cfg = entry_to_cfg(it->second, march_extent(kind, grid));
    switch (kind) {
        case TuneKind::Forward: return tile_supported(*cfg, dt);
        case TuneKind::Adjoint: return adjoint_tile_supported(*cfg);
        case TuneKind::Tangent: return tangent_tile_supported(*cfg, dt);
        case TuneKind::Zfast: return zfast_tile_supported(*cfg, dt);
    }
    return false;
}

void store_tuned(TuneKind kind, const pw_grid *grid, pw_dtype dt, const TileCfg &cfg) {
    std::lock_guard<std::mutex> lk(g_mu);
    load_locked();
    const int64_t zext = march_extent(kind, grid);
    Entry e{cfg.px, cfg.ry, static_cast<int>((zext + cfg.zlen - 1) / cfg.zlen), cfg.wpb, cfg.depth, cfg.share, true};
    g_table[make_key(kind, grid, dt)] = e;
    save_locked();
}

}  // namespace pw

using namespace pw;

extern "C" {

pw_status pw_tune(const pw_grid *grid, pw_dtype dtype, int32_t flags, pw_tile *fwd_best, pw_tile *adj_best) {
    if (!grid) return fail(PW_ERR_INVALID_ARG, "grid is NULL");
    if (grid->nx < 1 || grid->ny < 1 || grid->nz < 1 || grid->halo < 1 || grid->nx > (1 << 24) ||
        grid->ny > (1 << 24) || grid->nz > (1 << 24) || grid->halo > 1024)
        return fail(PW_ERR_INVALID_ARG, "bad grid extent");
    int64_t es = 0;
    switch (dtype) {
        case PW_F32: es = 4; break;
        case PW_F64: es = 8; break;
        case PW_BF16: case PW_F16: es = 2; break;
        default: return fail(PW_ERR_INVALID_ARG, "unknown dtype %d", static_cast<int>(dtype));
    }
    const int32_t all = PW_TUNE_FORWARD | PW_TUNE_ADJOINT | PW_TUNE_TANGENT;
    if (flags & ~(all | PW_TUNE_ZFAST)) return fail(PW_ERR_INVALID_ARG, "unknown flags 0x%x", flags);
    if (flags == 0) flags = all;
    const bool do_zf = flags & PW_TUNE_ZFAST;
    const bool full = dtype == PW_F32 || dtype == PW_F64;   // adjoint and tangent storage types
    const bool do_fwd = flags & PW_TUNE_FORWARD;
    const bool do_adj = (flags & PW_TUNE_ADJOINT) && full;
    const bool do_tan = (flags & PW_TUNE_TANGENT) && full;
    const int64_t cs = dtype == PW_F64 ? 8 : 4;
    const int64_t px = grid->nx + 2 * grid->halo, py = grid->ny + 2 * grid->halo, pz = grid->nz + 2 * grid->halo;
    const int64_t npad = px * py * pz, nint = grid->nx * grid->ny * grid->nz;
    if (px * py * cs >= (int64_t(1) << 31)) return fail(PW_ERR_UNSUPPORTED, "a z-plane larger than 2 GiB");
    if (do_zf && py * pz * cs >= (int64_t(1) << 31)) return fail(PW_ERR_UNSUPPORTED, "an x-plane larger than 2 GiB");
    int n = 0;
    if (hipGetDeviceCount(&n) != hipSuccess || n < 1) {
        (void)hipGetLastError();
        return fail(PW_ERR_NO_DEVICE, "no usable HIP device");
    }

    // Buffer sets of one launch's operands (inputs, direction, outputs or
    // gradients), enough of them to span about 1 GiB so that timed repeats
    // come from HBM, not from the MALL.
    const int64_t in_b = 3 * npad * es, out_b = 3 * (do_adj ? npad : nint) * cs, dir_b = do_tan ? 3 * npad * cs : 0;
    const int64_t set_b = in_b + out_b + dir_b;
    int64_t nsets = ((int64_t(1) << 30) + set_b - 1) / set_b;
    if (nsets < 1) nsets = 1;
    if (nsets > 8) nsets = 8;
    DevBuf in, out, dir, coef;
    if (in.alloc(size_t(nsets * in_b)) != hipSuccess || out.alloc(size_t(nsets * out_b)) != hipSuccess ||
        (dir_b && dir.alloc(size_t(nsets * dir_b)) != hipSuccess) ||
        coef.alloc(size_t(4 * grid->nz * cs)) != hipSuccess) {
        (void)hipGetLastError();
        return fail(PW_ERR_ALLOC, "scratch allocation for tuning failed");
    }
    hipStream_t s;
    if (hipStreamCreate(&s) != hipSuccess) return hip_fail(hipGetLastError(), "hipStreamCreate");
    // timing inputs at the workloads' scales (kernel times depend on the
    // data): winds in [-10, 10), which also serve as the adjoint's
    // cotangents, tangent directions in [-1, 1), coefficients in
    // [0.0025, 0.0075)
    const pw_dtype cdt = dtype == PW_F64 ? PW_F64 : PW_F32;
    hipError_t me = fill_tuning_data(in.p, nsets * 3 * npad, dtype, 1u, -10.f, 10.f, s);
    if (me == hipSuccess) me = hipMemsetAsync(out.p, 0, size_t(nsets * out_b), s);
    if (me == hipSuccess && dir_b) me = fill_tuning_data(dir.p, nsets * 3 * npad, cdt, 2u, -1.f, 1.f, s);
    if (me == hipSuccess) me = fill_tuning_data(coef.p, 4 * grid->nz, cdt, 3u, 0.0025f, 0.0075f, s);
    if (me != hipSuccess) {
        (void)hipStreamDestroy(s);
        return hip_fail(me, "scratch clear");
    }
    char *cb = static_cast<char *>(coef.p);
    auto fwd_args = [&](int64_t set) {
        char *ib = static_cast<char *>(in.p) + set * in_b, *ob = static_cast<char *>(out.p) + set * out_b;
        FwdArgs a;
        a.u = ib; a.v = ib + npad * es; a.w = ib + 2 * npad * es;
        a.su = ob; a.sv = ob + nint * cs; a.sw = ob + 2 * nint * cs;
        a.tzc1 = cb; a.tzc2 = cb + grid->nz * cs; a.tzd1 = cb + 2 * grid->nz * cs; a.tzd2 = cb + 3 * grid->nz * cs;
        a.tcx = a.tcy = 0.0025;
        a.nx = grid->nx; a.ny = grid->ny; a.nz = grid->nz; a.h = grid->halo;
        a.in_sy = px; a.in_sz = px * py; a.out_sy = grid->nx; a.out_sz = grid->nx * grid->ny;
        a.in_bytes = es;
        a.out_bytes = cs;
        return a;
    };
    // candidate shapes: columns per lane x rows per strip x z-chunks x waves per group
    auto candidates = [&](std::initializer_list<int> pxs, std::initializer_list<int> rys, int64_t zext,
                          bool (*ok)(const TileCfg &, pw_dtype), int max_depth) {
        std::vector<TileCfg> cands;
        for (int pxl : pxs)
            for (int ry : rys)
                for (int nzc : {1, 2, 3, 4, 6, 8})
                    for (int wpb : {1, 4})
                        for (int depth = 1; depth <= max_depth; ++depth) {
                            TileCfg c;
                            c.px = pxl;
                            c.ry = ry;
                            c.wpb = wpb;
                            c.depth = depth;
                            c.zlen = static_cast<int>((zext + nzc - 1) / nzc);
                            if (!ok(c, dtype) || (nzc > 1 && c.zlen < 4)) continue;
                            cands.push_back(c);
                        }
        return cands;
    };

    pw_status st = PW_OK;
    if (do_fwd) {
        auto cands = candidates({1, 2, 4}, {1, 2, 4}, grid->nz, &tile_supported, 2);
        // workgroups whose wavefronts share their edge rows through LDS
        for (int pxl : {2, 4, 8})
            for (int ry : {1, 2, 4})
                for (int nzc : {1, 2, 3, 4, 6, 8})
                    for (int wpb : {2, 4})
                        for (int share : {1, 2}) {
                            TileCfg c;
                            c.px = pxl;
                            c.ry = ry;
                            c.wpb = wpb;
                            c.depth = 1;
                            c.share = share;
                            c.zlen = static_cast<int>((grid->nz + nzc - 1) / nzc);
                            if (!tile_supported(c, dtype) || (nzc > 1 && c.zlen < 4)) continue;
                            cands.push_back(c);
                        }
        TileCfg bestc = default_forward_tile(fwd_args(0), dtype);
        st = pick_fastest(
            cands, [&](const TileCfg &c, int rep) { return launch_forward(fwd_args(rep % nsets), dtype, c, s); }, s,
            &bestc);
        if (st == PW_OK) {
            store_tuned(TuneKind::Forward, grid, dtype, bestc);
            if (fwd_best) *fwd_best = to_tile(bestc);
        }
    }
    if (st == PW_OK && do_adj) {
        auto adj_args = [&](int64_t set) {
            const FwdArgs a = fwd_args(set);
            AdjArgs g;
            g.u = a.u; g.v = a.v; g.w = a.w;
            g.gsu = a.u; g.gsv = a.v; g.gsw = a.w;   // cotangents: the zeroed inputs, read as interior arrays
            char *gb = static_cast<char *>(out.p) + set * out_b;
            g.gu = gb; g.gv = gb + npad * cs; g.gw = gb + 2 * npad * cs;
            g.tzc1 = a.tzc1; g.tzc2 = a.tzc2; g.tzd1 = a.tzd1; g.tzd2 = a.tzd2;
            g.tcx = g.tcy = 0.0025;
            g.nx = a.nx; g.ny = a.ny; g.nz = a.nz; g.h = a.h;
            g.in_sy = a.in_sy; g.in_sz = a.in_sz; g.out_sy = a.out_sy; g.out_sz = a.out_sz;
            return g;
        };
        auto ok = [](const TileCfg &c, pw_dtype) { return adjoint_tile_supported(c); };
        const auto cands = candidates({1}, {1, 2, 4}, pz, +ok, 2);
        TileCfg bestc = default_adjoint_tile(adj_args(0), dtype);
        st = pick_fastest(
            cands, [&](const TileCfg &c, int rep) { return launch_adjoint(adj_args(rep % nsets), dtype, c, s); }, s,
            &bestc);
        if (st == PW_OK) {
            store_tuned(TuneKind::Adjoint, grid, dtype, bestc);
            if (adj_best) *adj_best = to_tile(bestc);
        }
    }
    if (st == PW_OK && do_tan) {
        auto tan_args = [&](int64_t set) {
            TanArgs t;
            t.f = fwd_args(set);
            char *db = static_cast<char *>(dir.p) + set * dir_b;
            t.du = db; t.dv = db + npad * cs; t.dw = db + 2 * npad * cs;
            return t;
        };
        const auto cands = candidates({1, 2}, {1, 2}, grid->nz, &tangent_tile_supported, 2);
        TileCfg bestc = default_tangent_tile(tan_args(0), dtype);
        st = pick_fastest(
            cands, [&](const TileCfg &c, int rep) { return launch_tangent(tan_args(rep % nsets), dtype, c, s); }, s,
            &bestc);
        if (st == PW_OK) store_tuned(TuneKind::Tangent, grid, dtype, bestc);
    }
    if (st == PW_OK && do_zf) {
        // the same buffers read as z-fastest arrays (dense strides)
        auto zf_args = [&](int64_t set) {
            FwdArgs a = fwd_args(set);
            a.in_sy = pz; a.in_sz = py * pz; a.out_sy = grid->nz; a.out_sz = grid->ny * grid->nz;
            return a;
        };
        const auto cands = candidates({1, 2, 4}, {1, 2, 4, 8}, grid->nx, &zfast_tile_supported, 2);
        TileCfg bestc = default_zfast_tile(zf_args(0), dtype);
        st = pick_fastest(
            cands, [&](const TileCfg &c, int rep) { return launch_zfast(zf_args(rep % nsets), dtype, c, s); }, s,
            &bestc);
        if (st == PW_OK) store_tuned(TuneKind::Zfast, grid, dtype, bestc);
    }
    const hipError_t se = hipStreamSynchronize(s);
    (void)hipStreamDestroy(s);
    if (st != PW_OK) return st;
    return hip_fail(se, "tuning run");
}

pw_status pw_launch_shape(pw_kernel kind, const pw_grid *grid, pw_dtype dtype, pw_tile *out) {
    if (!grid || !out) return fail(PW_ERR_INVALID_ARG, "grid or out is NULL");
    if (grid->nx < 1 || grid->ny < 1 || grid->nz < 1 || grid->halo < 1)
        return fail(PW_ERR_INVALID_ARG, "bad grid extent");
    TuneKind k;
    switch (kind) {
        case PW_KERNEL_FORWARD: k = TuneKind::Forward; break;
        case PW_KERNEL_ADJOINT: k = TuneKind::Adjoint; break;
        case PW_KERNEL_TANGENT: k = TuneKind::Tangent; break;
        case PW_KERNEL_ZFAST: k = TuneKind::Zfast; break;
        default: return fail(PW_ERR_INVALID_ARG, "unknown kernel kind %d", static_cast<int>(kind));
    }
    if (dtype != PW_F32 && dtype != PW_F64 && dtype != PW_BF16 && dtype != PW_F16)
        return fail(PW_ERR_INVALID_ARG, "unknown dtype %d", static_cast<int>(dtype));
    if ((k == TuneKind::Adjoint || k == TuneKind::Tangent) && dtype != PW_F32 && dtype != PW_F64)
        return fail(PW_ERR_UNSUPPORTED, "the adjoint and tangent support PW_F32 and PW_F64 only");
    if (k == TuneKind::Forward) {   // PWADV_TILE takes precedence for the forward
        pw_tile t;
        const int e = env_forward_tile(&t);
        if (e < 0) return fail(PW_ERR_INVALID_ARG, "PWADV_TILE=\"%s\" is not a launch shape", std::getenv("PWADV_TILE"));
        if (e > 0) {
            TileCfg c = to_cfg(t);
            if (!tile_supported(c, dtype))
                return fail(PW_ERR_INVALID_ARG, "PWADV_TILE=\"%s\" is not a forward shape for this storage type",
                            std::getenv("PWADV_TILE"));
            *out = to_tile(c);
            return PW_OK;
        }
    }
    TileCfg c;
    if (!lookup_tuned(k, grid, dtype, &c)) {
        const int64_t px = grid->nx + 2 * grid->halo, py = grid->ny + 2 * grid->halo;
        FwdArgs a;
        a.nx = grid->nx; a.ny = grid->ny; a.nz = grid->nz; a.h = grid->halo;
        a.in_sy = px; a.in_sz = px * py; a.out_sy = grid->nx; a.out_sz = grid->nx * grid->ny;
        if (k == TuneKind::Forward) {
            c = default_forward_tile(a, dtype);
        } else if (k == TuneKind::Zfast) {
            c = default_zfast_tile(a, dtype);
        } else if (k == TuneKind::Tangent) {
            TanArgs t;
            t.f = a;
            c = default_tangent_tile(t, dtype);
        } else {
            AdjArgs g;
            g.nx = a.nx; g.ny = a.ny; g.nz = a.nz; g.h = a.h;
            g.in_sy = a.in_sy; g.in_sz = a.in_sz; g.out_sy = a.out_sy; g.out_sz = a.out_sz;
            c = default_adjoint_tile(g, dtype);
        }
    }
    *out = to_tile(c);
    return PW_OK;
}

pw_status pw_tune_reset(void) {
    std::lock_guard<std::mutex> lk(g_mu);
    g_table.clear();
    g_loaded = true;   // neither the built-in entries nor the file come back
    return PW_OK;
}

}  // extern "C"
