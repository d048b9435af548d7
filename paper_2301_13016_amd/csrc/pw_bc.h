// Boundary rules by addressing, for the forward and the adjoint kernels: where
// a read of a halo cell goes, and what its rule does to the value.
#pragma once

#include "pw_internal.h"

namespace pw {

// Padded index that a read of padded index p (0 <= p < n+2h) uses on an axis
// of n interior cells and halo h: p itself (an interior cell, or the stored
// halo under KEEP), or for a halo cell its source under the periodic or
// zero-gradient rule -- for the cells the depth-one stencil reads (p = h-1,
// p = n+h) the same map as the halo fill's, and in bounds for every p.
// Selects only, no branches: a branch between loads in flight would make the
// compiler wait for all of them where the paths join.
__device__ __forceinline__ int bc_src(int p, int n, int h, int mode) {
    const bool lo = p < h, hi = p >= n + h;
    const int per = lo ? p + n : (hi ? p - n : p);
    const int cpy = lo ? h : (hi ? n + h - 1 : p);
    return mode == PW_HALO_PERIODIC ? per : (mode == PW_HALO_COPY ? cpy : p);
}
// bc_src when the kernel is built for boundary rules (Bc), else p unchanged:
// the plain kernels carry no mapping code at all.
template <int Bc> __device__ __forceinline__ int bc_map(int p, int n, int h, int mode) {
    if constexpr (Bc) {
        return bc_src(p, n, h, mode);
    } else {
        (void)n;
        (void)h;
        (void)mode;
        return p;
    }
}

// Value rules by addressing (Bc == 2).  A halo cell's value is its source's
// value passed through one code per axis, in the halo fill's order x, y, z:
// 0 keeps it, 1 negates it (REFLECT_NEG), 2 replaces it by +0 (ZERO).  A code
// describing several axes has bit 1 = zero, bit 0 = negate: a zero drops
// what came before and a later negation turns it into -0, as the sequential
// fill does.  Codes of the three fields sit side by side, two bits each.
__device__ __forceinline__ uint32_t bc_compose(uint32_t first, uint32_t then) {   // one field
    return (then & 2u) ? then : (first ^ then);
}
__device__ __forceinline__ uint32_t bc_compose3(uint32_t first, uint32_t then) {  // three fields
    uint32_t z = then & 0x2Au;
    z |= z >> 1;   // both bits of every field whose later code zeroes
    return (then & z) | ((first ^ then) & ~z);
}
// Codes (three fields) of axis d for padded index p on an axis of n cells.
template <int Bc>
__device__ __forceinline__ uint32_t bc_axis_code(const uint32_t bcv, int d, int p, int n, int h) {
    if constexpr (Bc == 2) {
        const bool halo = p < h || p >= n + h;
        return halo ? (bcv >> (8 * d)) & 0x3Fu : 0u;
    } else {
        (void)bcv;
        (void)d;
        (void)p;
        (void)n;
        (void)h;
        return 0u;
    }
}

}  // namespace pw
