// Factored 27-point stencils of FP64 fields in z-marches, one barrier per
// plane: the adjoint's transposed stencils and the FP64 solid-mask stencils.
#pragma once

#include "lbfe_zring.h"

namespace lbfe {
namespace {

// The isotropic D3Q27 stencils factor into D1Q3 pieces (weights 1/6, 2/3, 1/6
// along each axis), so each one is an in-plane part read from one LDS plane
// and a z part over a register ring that a thread keeps for its column:
//   sum_i w_i g(x + c_i) = Wz (Wx Wy g),   3 sum_i w_i c_ix g(x + c_i) =
//   1/2 Wz (Dx Wy g),  ... y: 1/2 Wz (Wx Dy g),  ... z: 1/2 Dz (Wx Wy g).
constexpr double A1 = 1.0 / 6.0, A0 = 2.0 / 3.0;

// Wx Wy g at index c of an LDS plane with row stride W
template <int W> __device__ inline double smooth2(const double *g, int c) {
    const double r0 = A1 * g[c - W - 1] + A0 * g[c - W] + A1 * g[c - W + 1];
    const double r1 = A1 * g[c - 1] + A0 * g[c] + A1 * g[c + 1];
    const double r2 = A1 * g[c + W - 1] + A0 * g[c + W] + A1 * g[c + W + 1];
    return A1 * r0 + A0 * r1 + A1 * r2;
}
// Dx Wy g and Wx Dy g
template <int W> __device__ inline double dx_wy(const double *g, int c) {
    return A1 * (g[c - W + 1] - g[c - W - 1]) + A0 * (g[c + 1] - g[c - 1]) + A1 * (g[c + W + 1] - g[c + W - 1]);
}
template <int W> __device__ inline double wx_dy(const double *g, int c) {
    return A1 * (g[c + W - 1] - g[c - W - 1]) + A0 * (g[c + W] - g[c - W]) + A1 * (g[c + W + 1] - g[c - W + 1]);
}
__device__ inline double wz(double a, double b, double c) { return A1 * a + A0 * b + A1 * c; }
// the three in-plane parts of one plane, and the ring of the last two
struct Part3 {
    double x, y, z;
};
struct Ring3 {
    Part3 a{0, 0, 0}, b{0, 0, 0};  // two planes back, one plane back
    __device__ void push(const Part3 &n) {
        a = b;
        b = n;
    }
};

// Tile and chunk of this workgroup: each XCD takes a contiguous range of
// (chunk, tile) pairs, the tiles of one chunk consecutively, so that
// neighbouring tiles find each other's halo lines in that XCD's L2.
__device__ inline void xcd_tile(int &tile, int &chunk) {
    const unsigned nt = gridDim.x, nb = gridDim.x * gridDim.y, hw = blockIdx.y * gridDim.x + blockIdx.x;
    const unsigned q = nb >> 3, rem = nb & 7u, x = hw & 7u;
    const unsigned lid = x * q + (x < rem ? x : rem) + (hw >> 3);
    tile = (int)(lid % nt);
    chunk = (int)(lid / nt);
}

// Branch-free access to one plane of a field (masked lanes carry kNone: they
// read 0 and store nothing).
constexpr unsigned kNone = 0x80000000u;
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
__device__ inline __amdgpu_buffer_rsrc_t plane_of(const void *p, size_t first, unsigned plane, unsigned esize) {
    return __builtin_amdgcn_make_buffer_rsrc((char *)const_cast<void *>(p) + first * esize, 0, (int)(plane * esize),
                                             0x00020000);
}
__device__ inline void pld(double &v, __amdgpu_buffer_rsrc_t r, unsigned o) {
    v = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, o == kNone ? kNone : o * 8u, 0, 0));
}
__device__ inline void pld(float &v, __amdgpu_buffer_rsrc_t r, unsigned o) {
    v = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, o == kNone ? kNone : o * 4u, 0, 0));
}
__device__ inline void pst(double v, __amdgpu_buffer_rsrc_t r, unsigned o) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, o == kNone ? kNone : o * 8u, 0, 0);
}
__device__ inline void pst_nt(double v, __amdgpu_buffer_rsrc_t r, unsigned o) {  // non-temporal (policy bit 2)
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, o == kNone ? kNone : o * 8u, 0, 2);
}
__device__ inline void pst(float v, __amdgpu_buffer_rsrc_t r, unsigned o) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, o == kNone ? kNone : o * 4u, 0, 0);
}

// Planes per workgroup of these marches: `slots` workgroups run at
// once, each paying `fill` planes; the chunk from 64 down to 1 that minimises
// the busiest slot's plane iterations (the longer on ties).
inline int march_chunk(size_t tiles, int nz, size_t slots, int fill) {
    auto iters = [&](int c) { return (tiles * ((nz + c - 1) / c) + slots - 1) / slots * (size_t)(c + fill); };
    int cz = 64;
    for (int c = 63; c >= 1; --c)
        if (iters(c) < iters(cz)) cz = c;
    return cz;
}

}  // namespace
}  // namespace lbfe
