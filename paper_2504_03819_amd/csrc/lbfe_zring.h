// z-marching LDS ring for 27-point stencils of one scalar field, summed point by
// point: the solid-mask path's stencils of the FP32 and FP16 forms.
#pragma once

#include "lbfe_internal.h"

namespace lbfe {
namespace {

// ---------------------------------------------------------------------------
// z-marching stencil tiles.  A workgroup owns a 32 x 16 column tile of one
// z-chunk.  The field on four consecutive planes (tile + one-node
// halo) sits in an LDS ring; plane k+2 is loaded into
// registers while plane k is evaluated, so one barrier per plane suffices
// (the slot written at plane k+1 was last read at plane k-2).  Plane indices
// wrap periodically.
// ---------------------------------------------------------------------------
constexpr int ZTX = 32, ZTY = 16, ZWX = ZTX + 2, ZNR = ZWX * (ZTY + 2), ZCB = ZTX * ZTY;
constexpr int ZM = (ZNR + ZCB - 1) / ZCB;  // halo-region points per thread

__device__ inline int zwrap(int v, int n) {
    v %= n;
    return v < 0 ? v + n : v;
}

struct ZRing {
    double (*lds)[ZNR];  // [4][ZNR]
    const double *src;
    int a, b, tid, nz;
    bool own;       // the tile point is inside the grid
    unsigned node;  // its in-plane index
    unsigned plane;
    unsigned off[ZM];
    bool has[ZM];
    double pre[ZM];

    __device__ void init(const KP &k, double (*l)[ZNR], const double *field, int x0, int y0) {
        lds = l;
        src = field;
        tid = threadIdx.x;
        a = tid % ZTX;
        b = tid / ZTX;
        nz = k.nz;
        plane = k.plane;
        own = x0 + a < k.nx && y0 + b < k.ny;
        node = own ? (unsigned)(y0 + b) * k.nx + (x0 + a) : 0u;
#pragma unroll
        for (int m = 0; m < ZM; ++m) {
            const int r = tid + m * ZCB;
            has[m] = r < ZNR;
            const int rr = has[m] ? r : 0;
            off[m] = (unsigned)zwrap(y0 + rr / ZWX - 1, k.ny) * k.nx + zwrap(x0 + rr % ZWX - 1, k.nx);
        }
    }
    __device__ void load(int p) {
        const size_t base = (size_t)zwrap(p, nz) * plane;
#pragma unroll
        for (int m = 0; m < ZM; ++m)
            if (has[m]) pre[m] = src[base + off[m]];
    }
    __device__ void commit(int p) {
#pragma unroll
        for (int m = 0; m < ZM; ++m)
            if (has[m]) lds[p & 3][tid + m * ZCB] = pre[m];
    }
    // the field at (x + dx, y + dy, plane p)
    __device__ double at(int p, int dx, int dy) const { return lds[p & 3][(b + 1 + dy) * ZWX + a + 1 + dx]; }
    // planes [zs, ze) of the chunk, body(k) once per plane after the barrier
    template <class Body> __device__ void march(int zs, int ze, Body body) {
        load(zs - 1);
        commit(zs - 1);
        load(zs);
        commit(zs);
        load(zs + 1);
        for (int k = zs; k < ze; ++k) {
            commit(k + 1);
            __syncthreads();
            if (k + 1 < ze) load(k + 2);
            body(k);
        }
    }
};

__device__ inline void ztile(const KP &kp, int cz, int &x0, int &y0, int &zs, int &ze) {
    const int ntx = (kp.nx + ZTX - 1) / ZTX;
    x0 = (int)(blockIdx.x % ntx) * ZTX;
    y0 = (int)(blockIdx.x / ntx) * ZTY;
    zs = (int)blockIdx.y * cz;
    ze = min(zs + cz, kp.nz);
}

// Grid of the z-marching kernels.
constexpr int kZChunk = 16;
dim3 zgrid(const KP &kp) {
    const unsigned ntx = (kp.nx + ZTX - 1) / ZTX, nty = (kp.ny + ZTY - 1) / ZTY;
    return dim3(ntx * nty, (unsigned)((kp.nz + kZChunk - 1) / kZChunk));
}

}  // namespace
}  // namespace lbfe
