// Forward Piacsek-Williams advection: launch dispatch, launch-shape rules and
// defaults, and the bandwidth-calibration copy kernels.  The stencil kernel
// itself is in pw_forward_impl.h (instantiated per storage type in
// pw_forward_{f32,f64,bf16,f16}.hip).
#include "pw_internal.h"

namespace pw {
namespace {

// Plain device copy, 16 bytes per lane per step, grid-stride.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void copy16_kernel(const u32x4 *__restrict__ src, u32x4 *__restrict__ dst,
                                                     int64_t n) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) {
        u32x4 x = __builtin_nontemporal_load(src + i);
        __builtin_nontemporal_store(x, dst + i);
    }
}

// Three copies in one grid-stride loop: the stencil's traffic pattern (three
// arrays read, three written) without the stencil.
__global__ __launch_bounds__(256) void copy16x3_kernel(const u32x4 *__restrict__ a, const u32x4 *__restrict__ b,
                                                       const u32x4 *__restrict__ c, u32x4 *__restrict__ x,
                                                       u32x4 *__restrict__ y, u32x4 *__restrict__ z, int64_t n) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) {
        const u32x4 p = __builtin_nontemporal_load(a + i);
        const u32x4 q = __builtin_nontemporal_load(b + i);
        const u32x4 r = __builtin_nontemporal_load(c + i);
        __builtin_nontemporal_store(p, x + i);
        __builtin_nontemporal_store(q, y + i);
        __builtin_nontemporal_store(r, z + i);
    }
}

// Calibration probe: Mode 0 copies, 1 only reads (an XOR of everything read
// is stored to sink only if it equals a fixed pattern, so that the loads are
// kept), 2 only writes.  Each lane issues L independent 16-byte loads before
// their stores; grid-stride over n vectors.  NtL / NtS: non-temporal loads /
// stores.
template <int L, bool NtL, bool NtS, int Mode>
__global__ __launch_bounds__(256) void probe_kernel(const u32x4 *__restrict__ src, u32x4 *__restrict__ dst,
                                                    int64_t n, u32x4 *__restrict__ sink) {
    const int64_t step = static_cast<int64_t>(gridDim.x) * 256 * L;
    u32x4 acc = {0u, 0u, 0u, 0u};
    for (int64_t base = static_cast<int64_t>(blockIdx.x) * 256 * L; base < n; base += step) {
        u32x4 x[L];
#pragma unroll
        for (int l = 0; l < L; ++l) {
            const int64_t i = base + l * 256 + threadIdx.x;
            if constexpr (Mode == 2) {
                x[l] = u32x4{static_cast<unsigned>(i), 1u, 2u, 3u};
            } else if (i < n) {
                x[l] = NtL ? __builtin_nontemporal_load(src + i) : src[i];
            } else {
                x[l] = acc;
            }
        }
#pragma unroll
        for (int l = 0; l < L; ++l) {
            const int64_t i = base + l * 256 + threadIdx.x;
            if constexpr (Mode == 1) {
                acc ^= x[l];
            } else if (i < n) {
                if constexpr (NtS)
                    __builtin_nontemporal_store(x[l], dst + i);
                else
                    dst[i] = x[l];
            }
        }
    }
    if constexpr (Mode == 1) {
        if (acc.x == 0x9e3779b9u && acc.y == 0x7f4a7c15u && acc.z == 0x85ebca6bu && acc.w == 0xc2b2ae35u)
            sink[threadIdx.x] = acc;
    }
}

template <int L, int Mode>
void launch_probe_l(int flags, dim3 g, hipStream_t s, const u32x4 *src, u32x4 *dst, int64_t n, u32x4 *sink) {
    switch (flags & 3) {
        case 0: hipLaunchKernelGGL((probe_kernel<L, false, false, Mode>), g, dim3(256), 0, s, src, dst, n, sink); break;
        case 1: hipLaunchKernelGGL((probe_kernel<L, true, false, Mode>), g, dim3(256), 0, s, src, dst, n, sink); break;
        case 2: hipLaunchKernelGGL((probe_kernel<L, false, true, Mode>), g, dim3(256), 0, s, src, dst, n, sink); break;
        default: hipLaunchKernelGGL((probe_kernel<L, true, true, Mode>), g, dim3(256), 0, s, src, dst, n, sink); break;
    }
}

template <int Mode>
void launch_probe_m(int loads, int flags, dim3 g, hipStream_t s, const u32x4 *src, u32x4 *dst, int64_t n,
                    u32x4 *sink) {
    switch (loads) {
        case 1: launch_probe_l<1, Mode>(flags, g, s, src, dst, n, sink); break;
        case 2: launch_probe_l<2, Mode>(flags, g, s, src, dst, n, sink); break;
        case 4: launch_probe_l<4, Mode>(flags, g, s, src, dst, n, sink); break;
        default: launch_probe_l<8, Mode>(flags, g, s, src, dst, n, sink); break;
    }
}

}  // namespace

pw_status launch_probe(int mode, int loads, int flags, const void *src, void *dst, int64_t nbytes, int blocks,
                       hipStream_t s) {
    const int64_t n = nbytes / 16;
    const dim3 g(static_cast<unsigned>(blocks));
    const u32x4 *sp = static_cast<const u32x4 *>(src);
    u32x4 *dp = static_cast<u32x4 *>(dst);
    switch (mode) {
        case 0: launch_probe_m<0>(loads, flags, g, s, sp, dp, n, dp); break;
        case 1: launch_probe_m<1>(loads, flags, g, s, sp, nullptr, n, dp); break;
        default: launch_probe_m<2>(loads, flags, g, s, nullptr, dp, n, dp); break;
    }
    return hip_fail(hipGetLastError(), "stream probe launch");
}

// Shapes instantiated with rows shared through LDS (pw_forward_lds_*.hip).
bool shared_tile_supported(const TileCfg &c, pw_dtype dt) {
    if ((c.share != 1 && c.share != 2) || (c.wpb != 2 && c.wpb != 4) || c.depth != 1 || c.zlen < 1) return false;
    switch (dt) {
        case PW_F32: return c.px == 4 && (c.ry == 1 || c.ry == 2 || c.ry == 4);
        case PW_BF16:
        case PW_F16: return (c.px == 4 && (c.ry == 2 || c.ry == 4)) || (c.px == 8 && c.ry == 2);
        case PW_F64: return c.px == 2 && (c.ry == 2 || c.ry == 4);
    }
    return false;
}

bool tile_supported(const TileCfg &c, pw_dtype dt) {
    if (c.share != 0) return shared_tile_supported(c, dt);
    if (c.zlen < 1 || c.wpb < 1 || c.wpb > 8 || (c.depth != 1 && c.depth != 2)) return false;
    const bool half = dt == PW_BF16 || dt == PW_F16;
    if (dt == PW_F64) return (c.px == 1 || c.px == 2) && (c.ry == 1 || c.ry == 2 || c.ry == 4);
    if (c.px == 8) return half && (c.ry == 1 || c.ry == 2);
    if (c.px == 4) return c.ry == 1 || c.ry == 2 || c.ry == 4;
    return (c.px == 1 || c.px == 2) && (c.ry == 1 || c.ry == 2 || c.ry == 4);
}

TileCfg default_forward_tile(const FwdArgs &a, pw_dtype dt) {
    // Narrow and ragged grids: one column per lane, packed where that makes
    // fewer strips (see strip_march_t): against the shapes that plain strips
    // made cheapest FP32 267x185x66 31.3 -> 25.3 us, 337x713x26 46.4 -> 40.4,
    // BF16 78x230x187 29.8 -> 23.1.  Wide ones: 16 bytes per lane with shared
    // rows -- a short workgroup (two wavefronts of one row, FP32) while the grid
    // is small enough that wavefronts in flight decide, tall ones (four
    // wavefronts of two rows, half the rows read twice) where the bytes do.
    const int64_t pts = a.nx * a.ny * a.nz;
    const bool rules = has_rules(a);
    const auto pick = [&](const ShapeCost *s, int n) { return cheapest_shape(s, n, a.nx, a.ny, a.nz, !rules); };
    if (rules) {
        // One-column strips are not packed here, and strips at the x end cost
        // more (bc_patch_x; tall shared workgroups FP32 600x600x120 404 us, of
        // one row 281): lists of their own, fitted to 141 grids in FP32, 125 in
        // FP64 and 111 in BF16, 4, 4 and 5 % slower than the best shape.  The
        // lists below, whose packed strips do not run here, were 13, 9 and 18 %
        // slower: FP32 134x95x92 20.8 -> 17.8 us, 140x300x150 66.5 -> 53.9,
        // BF16 401x134x71 51.2 -> 32.0, FP64 136x767x21 53.1 -> 41.9.
        static const ShapeCost f32[] = {{1, 2, 1, 1, 0, 64, 2048, 1.00, 0.3}, {1, 4, 1, 1, 0, 64, 2048, 1.34, 3.3},
                                        {2, 2, 1, 1, 0, 128, 2048, 1.41, 0.5, 1.37},
                                        {4, 1, 1, 1, 0, 256, 2048, 1.40, 0.3, 1.12},
                                        {4, 1, 4, 1, 2, 256, 2048, 1.27, 1.7, 1.13},
                                        {4, 2, 4, 1, 2, 256, 1024, 1.15, 3.1, 2.35}};
        static const ShapeCost f64[] = {{1, 2, 1, 1, 0, 64, 2048, 1.00, 0.3}, {1, 4, 1, 1, 0, 64, 1024, 0.69, 5.0},
                                        {2, 2, 1, 1, 0, 128, 1024, 0.80, 1.0, 1.04},
                                        {2, 2, 4, 1, 2, 128, 1024, 0.65, 5.0, 1.82}};
        static const ShapeCost half[] = {{1, 2, 1, 1, 0, 64, 2048, 1.00, 0.3}, {1, 4, 1, 1, 0, 64, 2048, 1.67, 1.3},
                                         {2, 2, 1, 1, 0, 128, 2048, 1.66, 0.3}, {2, 4, 1, 1, 0, 128, 2048, 3.06, 1.0}};
        return dt == PW_F32 ? pick(f32, 6) : dt == PW_F64 ? pick(f64, 4) : pick(half, 4);
    }
    if (dt == PW_F32) {
        // 137 grids, 6 % slower than the best shape.  With a line at 16 M points
        // between the short and the tall shape, instead of the tall one's longer
        // start, 9 %: 512x512x60 81 us, tall 68; 500x500x63 88 / 79; 400x400x99
        // 104 / 94; 600x600x120 308 / 231.
        static const ShapeCost s[] = {{1, 2, 1, 1, 0, 64, 2048, 0.90}, {1, 4, 1, 1, 0, 64, 2048, 1.50},
                                      {4, 1, 2, 1, 2, 256, 2048, 0.95},
                                      {4, 2, 4, 1, 2, 256, 1024, 0.77, 4.8, 1.21}};
        return pick(s, 4);
    }
    if (dt == PW_F64) {
        // Two lists: a tall shape with too few wavefronts to fill the chip loses
        // (306x492x21, 3.2 M points: 44.8 us, one-row strips 33.9), and where they
        // do the others read more (250x250x100, 6.2 M: 65.3 us, two-row strips
        // 72.2); around 5 M points they are even (208x631x30 51.5 / 49.7,
        // 207x278x87 62.2 / 67.7).  84 grids below, 4 % slower than the best
        // shape (with one-column strips counted as plain ones 6 %), 53 above, 2 %.
        static const ShapeCost small[] = {{1, 2, 1, 1, 0, 64, 1024, 1.00, 0.5}, {2, 1, 1, 1, 0, 128, 1024, 0.55, 0.9},
                                          {2, 2, 1, 1, 0, 128, 1024, 0.93, 1.4}};
        static const ShapeCost large[] = {{1, 4, 1, 1, 0, 64, 1024, 1.30}, {2, 2, 4, 1, 2, 128, 1024, 1.00}};
        return pts < 5000000 ? pick(small, 3) : pick(large, 2);
    }
    // 16-bit storage: 165 grids, 7 % slower than the best shape.  The tallest
    // shape only where it fills its strips: BF16 512x512x60 64.6 us, two-row
    // strips 74.3; 900x700x100 308 / 322; 600x600x120 226 / 224.
    static const ShapeCost s[] = {{1, 2, 1, 1, 0, 64, 2048, 0.67}, {1, 4, 1, 1, 0, 64, 2048, 1.09},
                                  {2, 2, 1, 1, 0, 128, 2048, 0.97}, {4, 2, 2, 1, 1, 256, 2048, 1.58},
                                  {4, 4, 2, 1, 2, 256, 1024, 1.28, 4.8, 1.79}};
    return pick(s, 5);
}

pw_status launch_forward(const FwdArgs &a, pw_dtype dt, const TileCfg &cfg, hipStream_t s) {
    if (!tile_supported(cfg, dt)) return fail(PW_ERR_INVALID_ARG, "unsupported tile configuration");
    const bool bc = has_rules(a);
    if (bc && cfg.share == 0 && cfg.wpb > 4) {
        // boundary rules are built for up to four wavefronts per workgroup;
        // the strips are independent, so regrouping them changes no result
        TileCfg c = cfg;
        c.wpb = 4;
        return launch_forward(a, dt, c, s);
    }
    if (a.nx < cfg.px) {
        // a row narrower than one lane's columns: the vectors of the last
        // rows would run past the array (load_row needs rows of at least
        // PX - 1 elements, load_epi of PX); one-column lanes give the same bits
        TileCfg c = cfg;
        c.px = 1;
        c.share = 0;
        return launch_forward(a, dt, c, s);
    }
    if (cfg.share != 0) {
        switch (dt) {
            case PW_F32: return launch_forward_lds_f32(a, cfg, s);
            case PW_F64: return launch_forward_lds_f64(a, cfg, s);
            case PW_BF16: return launch_forward_lds_bf16(a, cfg, s);
            case PW_F16: return launch_forward_lds_f16(a, cfg, s);
        }
        return fail(PW_ERR_UNSUPPORTED, "dtype %d", static_cast<int>(dt));
    }
    switch (dt) {
        case PW_F32: return launch_forward_f32(a, cfg, s);
        case PW_F64: return launch_forward_f64(a, cfg, s);
        case PW_BF16: return launch_forward_bf16(a, cfg, s);
        case PW_F16: return launch_forward_f16(a, cfg, s);
    }
    return fail(PW_ERR_UNSUPPORTED, "dtype %d", static_cast<int>(dt));
}

pw_status launch_copy3(const void *const *src, void *const *dst, int64_t nbytes, hipStream_t s) {
    const int64_t n = nbytes / 16;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 8192) blocks = 8192;   // measured best for this pattern on MI355X
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(copy16x3_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s,
                       static_cast<const u32x4 *>(src[0]), static_cast<const u32x4 *>(src[1]),
                       static_cast<const u32x4 *>(src[2]), static_cast<u32x4 *>(dst[0]), static_cast<u32x4 *>(dst[1]),
                       static_cast<u32x4 *>(dst[2]), n);
    return hip_fail(hipGetLastError(), "three-stream copy kernel launch");
}

pw_status launch_copy(const void *src, void *dst, int64_t nbytes, hipStream_t s) {
    const int64_t n = nbytes / 16;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 256 * 16) blocks = 256 * 16;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(copy16_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s,
                       static_cast<const u32x4 *>(src), static_cast<u32x4 *>(dst), n);
    return hip_fail(hipGetLastError(), "copy kernel launch");
}

}  // namespace pw
