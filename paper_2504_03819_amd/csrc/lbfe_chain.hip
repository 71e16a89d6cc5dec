// The stencil chain of one step on gfx950:
//   rho  -> mu = mu0 - kappa lap_h rho                      (Eq. (32))
//           (mu0 = mu0(rho) per node comes from the pass that formed rho, on
//           large periodic grids it is formed here)
//        -> solid-node mu by the wall average              (Eq. (36))
//   mu   -> G = grad_h mu, F = (1/3 - rho) G,               (Eq. (12))
//           u = (j + F/2)/rho, phi = (p_m - rho/3) u
//   phi  -> Q_aa = -3 d_a phi_a                              (Eq. (27))
//
// The isotropic D3Q27 stencils factor into D1Q3 pieces (weights 1/6, 2/3, 1/6
// along each axis), so every stencil is evaluated as an in-plane part, read
// from one LDS plane, and a z part, combined in a three-plane register ring
// that each thread keeps for the columns it owns:
//   lap_h g = 6 (Wz (Wx Wy g) - g)
//   d_x g   = 1/2 Wz (Dx Wy g),  d_y g = 1/2 Wz (Wx Dy g),  d_z g = 1/2 Dz (Wx Wy g)
// with W the D1Q3 weights and D g = g(+1) - g(-1).  Three kernels sum in this
// order, so all of them give the same bits: k_chain_block for small grids,
// k_chain_march for large ones, k_wall_planes for mu of the solid planes of a
// large walled grid.  Outputs per fluid node: mu (double), F and Q (compute
// precision); mu is also written at the solid planes.
#include <type_traits>

#include "lbfe_device.h"

namespace lbfe {
namespace {

constexpr int TX = 64, TY = 16, NTC = TX * TY;  // 1024 threads, one workgroup per CU (LDS)
constexpr double A1 = 1.0 / 6.0, A0 = 2.0 / 3.0;       // D1Q3 weights

// Branch-free global access: raw buffer loads/stores through a descriptor
// of one plane; masked lanes use an offset past the plane, which the
// hardware drops (stores) or reads as zero (loads).  Keeping every global
// access outside lane-divergent branches lets the compiler count outstanding
// memory operations instead of draining them all at each plane.
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
constexpr unsigned kOOB = 0x80000000u;
__device__ inline __amdgpu_buffer_rsrc_t plane_rsrc(const void *base, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000);
}
// The outputs mu, F, Q are stored non-temporal (cache-policy bit 2): the
// collide pass reads them once, after the whole chain, and the L2 is left to
// the stencil halos.
constexpr int kStoreNT = 2;
__device__ inline void bstore(double v, __amdgpu_buffer_rsrc_t r, unsigned off) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, off, 0, kStoreNT);
}
__device__ inline void bstore(float v, __amdgpu_buffer_rsrc_t r, unsigned off) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, off, 0, kStoreNT);
}
__device__ inline void bload(double &v, __amdgpu_buffer_rsrc_t r, unsigned off) {
    v = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
__device__ inline void bload(float &v, __amdgpu_buffer_rsrc_t r, unsigned off) {
    v = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}

__device__ inline int wrap(int v, int n) {
    v %= n;
    return v < 0 ? v + n : v;
}

// Wx Wy g of the 3x3 in-plane neighbourhood of index c in a row-major LDS
// plane with row stride W.
template <int W> __device__ inline double smooth2(const double *g, int c) {
    const double r0 = A1 * g[c - W - 1] + A0 * g[c - W] + A1 * g[c - W + 1];
    const double r1 = A1 * g[c - 1] + A0 * g[c] + A1 * g[c + 1];
    const double r2 = A1 * g[c + W - 1] + A0 * g[c + W] + A1 * g[c + W + 1];
    return A1 * r0 + A0 * r1 + A1 * r2;
}

// In-plane parts of grad mu at index c of an LDS plane with row stride W:
// Dx Wy g, Wx Dy g, Wx Wy g.
template <int W> __device__ inline void plane_grad(const double *g, int c, double &Av, double &Bv, double &Cv) {
    const double l0 = g[c - W - 1], l1 = g[c - W], l2 = g[c - W + 1];
    const double m0 = g[c - 1], m1 = g[c], m2 = g[c + 1];
    const double h0 = g[c + W - 1], h1 = g[c + W], h2 = g[c + W + 1];
    Av = A1 * (l2 - l0) + A0 * (m2 - m0) + A1 * (h2 - h0);
    Bv = A1 * (h0 - l0) + A0 * (h1 - l1) + A1 * (h2 - l2);
    Cv = A1 * (A1 * l0 + A0 * l1 + A1 * l2) + A0 * (A1 * m0 + A0 * m1 + A1 * m2) +
         A1 * (A1 * h0 + A0 * h1 + A1 * h2);
}

// F and phi at a fluid node from the in-plane parts of grad mu in the planes
// below, at and above it, its density, mu and momentum.
template <class real>
__device__ inline void force_phi(double Aa, double Ab, double Ac, double Ba, double Bb, double Bc, double Ca, double Cc,
                                 double rd, double mu, const real (&j)[3], real &Fx, real &Fy, real &Fz,
                                 real (&phi)[3]) {
    const double gx = 0.5 * (A1 * Aa + A0 * Ab + A1 * Ac);
    const double gy = 0.5 * (A1 * Ba + A0 * Bb + A1 * Bc);
    const double gz = 0.5 * (Cc - Ca);
    const double c1 = 1.0 / 3.0 - rd;
    Fx = (real)(c1 * gx);
    Fy = (real)(c1 * gy);
    Fz = (real)(c1 * gz);
    const real ir = (real)1 / (real)rd;
    const real ux = (j[0] + (real)0.5 * Fx) * ir;
    const real uy = (j[1] + (real)0.5 * Fy) * ir;
    const real uz = (j[2] + (real)0.5 * Fz) * ir;
    // p_m - rho/3 with p_m = (1 + mu)/3
    const real c2 = (real)((1.0 + mu - rd) * (1.0 / 3.0));
    phi[0] = c2 * ux;
    phi[1] = c2 * uy;
    phi[2] = c2 * uz;
}

// In-plane parts of d_x phi_x, d_y phi_y, d_z phi_z at index c.
template <int W, class real>
__device__ inline void plane_div(const real *gx, const real *gy, const real *gz, int c, real &X, real &Y, real &Z) {
    const real w1r = (real)A1, w0r = (real)A0;
    X = w1r * (gx[c - W + 1] - gx[c - W - 1]) + w0r * (gx[c + 1] - gx[c - 1]) + w1r * (gx[c + W + 1] - gx[c + W - 1]);
    Y = w1r * (gy[c + W - 1] - gy[c - W - 1]) + w0r * (gy[c + W] - gy[c - W]) + w1r * (gy[c + W + 1] - gy[c - W + 1]);
    Z = w1r * (w1r * gz[c - W - 1] + w0r * gz[c - W] + w1r * gz[c - W + 1]) +
        w0r * (w1r * gz[c - 1] + w0r * gz[c] + w1r * gz[c + 1]) +
        w1r * (w1r * gz[c + W - 1] + w0r * gz[c + W] + w1r * gz[c + W + 1]);
}
// Q from the in-plane parts in the planes below, at and above the node.
template <class real>
__device__ inline void q_of(real Xa, real Xb, real Xc, real Ya, real Yb, real Yc, real Za, real Zc, real &qx, real &qy,
                            real &qz) {
    const real h = (real)(-1.5), w1r = (real)A1, w0r = (real)A0;
    qx = h * (w1r * Xa + w0r * Xb + w1r * Xc);
    qy = h * (w1r * Ya + w0r * Yb + w1r * Yc);
    qz = h * (Zc - Za);
}

// The R-row forms of smooth2, plane_grad and plane_div: R vertically adjacent
// points from index c of the first, the x parts of a row formed once for the
// (up to three) points that share it.  Every value is rounded as in the
// one-point form.
template <int W, int R> __device__ inline void smooth_rows(const double *g, int c, double (&P)[R], double (&mid)[R]) {
    double x[R + 2];
#pragma unroll
    for (int i = 0; i < R + 2; ++i) {
        const double *r = g + c + (i - 1) * W;
        const double l = r[-1], m = r[0], h = r[1];
        x[i] = A1 * l + A0 * m + A1 * h;
        if (i >= 1 && i <= R) mid[i - 1] = m;
    }
#pragma unroll
    for (int i = 0; i < R; ++i) P[i] = A1 * x[i] + A0 * x[i + 1] + A1 * x[i + 2];
}
template <int W, int R>
__device__ inline void grad_rows(const double *g, int c, double (&A)[R], double (&B)[R], double (&C)[R], double (&mid)[R]) {
    double l[R + 2], m[R + 2], h[R + 2], s[R + 2];
#pragma unroll
    for (int i = 0; i < R + 2; ++i) {
        const double *r = g + c + (i - 1) * W;
        l[i] = r[-1], m[i] = r[0], h[i] = r[1];
        s[i] = A1 * l[i] + A0 * m[i] + A1 * h[i];
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
        A[i] = A1 * (h[i] - l[i]) + A0 * (h[i + 1] - l[i + 1]) + A1 * (h[i + 2] - l[i + 2]);
        B[i] = A1 * (l[i + 2] - l[i]) + A0 * (m[i + 2] - m[i]) + A1 * (h[i + 2] - h[i]);
        C[i] = A1 * s[i] + A0 * s[i + 1] + A1 * s[i + 2];
        mid[i] = m[i + 1];
    }
}
template <int W, int R, class real>
__device__ inline void div_rows(const real *gx, const real *gy, const real *gz, int c, real (&X)[R], real (&Y)[R],
                                real (&Z)[R]) {
    const real w1r = (real)A1, w0r = (real)A0;
    real dx[R + 2], yl[R + 2], ym[R + 2], yh[R + 2], sz[R + 2];
#pragma unroll
    for (int i = 0; i < R + 2; ++i) {
        const int o = c + (i - 1) * W;
        dx[i] = gx[o + 1] - gx[o - 1];
        yl[i] = gy[o - 1], ym[i] = gy[o], yh[i] = gy[o + 1];
        sz[i] = w1r * gz[o - 1] + w0r * gz[o] + w1r * gz[o + 1];
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
        X[i] = w1r * dx[i] + w0r * dx[i + 1] + w1r * dx[i + 2];
        Y[i] = w1r * (yl[i + 2] - yl[i]) + w0r * (ym[i + 2] - ym[i]) + w1r * (yh[i + 2] - yh[i]);
        Z[i] = w1r * sz[i] + w0r * sz[i + 1] + w1r * sz[i + 2];
    }
}

// ---------------------------------------------------------------------------
// The march of large grids.  The three stencils run at the same time on
// planes one stage apart, each on waves of its own, so that a plane costs one
// barrier: at iteration t the five mu waves store rho(t) to LDS and evaluate
// mu(t-2), the seven phi waves F and phi(t-4), the four Q waves Q(t-6), each
// from what the iteration before left in LDS.  A thread owns 5, 3 or 4 points
// above one another and forms the x parts of a row once for all of them, and
// keeps only its own stage's rings (126 VGPRs at 16 waves; one thread that
// keeps all three needs 204).  rho stays in LDS for five planes, until phi has
// used it: read again from memory it had left the L2 (256^3: +13 % traffic).
// The planes zs-3 .. zs-1 are loaded at once, so a chunk of c planes takes
// c + 6 iterations, and fill planes that a stage does not need have an empty
// descriptor.  Bound by the halo and fill traffic (us, against the march with
// three barriers and one point per thread): 128^3 FP64 57 -> 47, FP32 42 ->
// 34; 192x192x96 83 -> 68, 62 -> 47; 512^3 2920 -> 2720-2870, 1955 -> 1743;
// 256^3 388 -> 418, 270 -> 246-275.  MU0: mu0(rho) is formed here instead of
// read (kp.mu0_in_chain).  WALLS: phi is zero on the solid planes, whose mu
// stands in mu0 (k_wall_planes).  Before, a march of its own formed the solid
// planes between walls (us with the wall density, before / now: FP64 128^3 63 /
// 54, 256^3 411 / 394; FP32 128^3 51 / 40, 192x192x96 67 / 54, 256^3 279 / 267; 211 x
// 187 x 150 112 / 117).
// ---------------------------------------------------------------------------
template <class real, bool MU0, bool WALLS>
__global__ __launch_bounds__(NTC) void k_chain_march(KP kp, const double *__restrict__ rho, const double *__restrict__ mu0,
                                               const void *jq, double *__restrict__ mu, void *Fq, void *Qq, int cz) {
    constexpr int HM = 2, HR = 3;  // halos of the mu and rho regions
    // rows per thread and waves of the mu, phi and Q roles
    constexpr int RB = 5, RC = 3, RD = 4, VB = 5, VC = 7, VD = 4;
    constexpr int WM = TX + 2 * HM, YM = TY + 2 * HM, BM = (YM + RB - 1) / RB;  // mu region, row blocks
    constexpr int WR = TX + 2 * HR, NR = WR * (TY + 2 * HR), NRP = WR * (BM * RB + 2);
    constexpr int WP = TX + 2, YP = TY + 2, BP = YP / RC;
    constexpr int MR = (NR + VB * 64 - 1) / (VB * 64);  // rho points per thread of the mu role
    static_assert((VB + VC + VD) * 64 == NTC && BM * WM <= VB * 64 && BP * RC == YP && BP * WP <= VC * 64 &&
                      TX * (TY / RD) == VD * 64,
                  "one unit per thread of a role");
    constexpr int LR = MR * VB * 64 > NRP ? MR * VB * 64 : NRP;  // whole rounds of the mu role's stores
    static_assert(NRP >= NR, "rho plane");
    __shared__ double sr[5][LR];               // rho plane t (slot t mod 5)
    __shared__ double sm[2][BM * RB * WM];     // mu plane
    __shared__ real sp[2][3][WP * YP];         // phi plane

    // Workgroups are dealt round-robin to the 8 XCDs in linear order; the
    // linear id is remapped so that each XCD runs a contiguous range of
    // (chunk, tile) pairs, tiles of one chunk consecutively: neighbouring
    // tiles then share their halo planes through that XCD's L2.
    const int ntx = (kp.nx + TX - 1) / TX;
    const unsigned ntiles = gridDim.x, nb = gridDim.x * gridDim.y;
    const unsigned hw = blockIdx.y * gridDim.x + blockIdx.x;
    const unsigned q = nb >> 3, rem = nb & 7u, xcd = hw & 7u;
    const unsigned lid = xcd * q + (xcd < rem ? xcd : rem) + (hw >> 3);
    const int tile = (int)(lid % ntiles), chunk = (int)(lid / ntiles);
    const int x0 = (tile % ntx) * TX, y0 = (tile / ntx) * TY;
    const int zs = kp.z0 + chunk * cz;
    const int ze = min(zs + cz, kp.z1);
    const size_t N = kp.N;
    constexpr unsigned S = sizeof(real);
    const unsigned pbytes8 = kp.plane * 8u, pbytesr = kp.plane * S;

    // plane indices wrap periodically; inside the march they advance by one
    auto next = [&](int g) { return g + 1 == kp.nz ? 0 : g + 1; };
    auto pbase = [&](int g) { return (size_t)g * kp.plane; };
    auto inside = [&](int x, int y) { return x >= 0 && x < TX && y >= 0 && y < TY && x0 + x < kp.nx && y0 + y < kp.ny; };
    auto node = [&](int x, int y) { return (unsigned)wrap(y0 + y, kp.ny) * kp.nx + (unsigned)wrap(x0 + x, kp.nx); };

    auto solid = [&](int g) { return WALLS && (g == 0 || g == kp.nz - 1); };

    const int tb = zs, te = ze + 5;  // first and last iteration
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (wave < VC) {
        // ---- F and phi(t-4) from the in-plane parts of mu(t-5 .. t-3)
        const int u = wave * 64 + lane, pa = u % WP, pb = u / WP * RC;
        const bool has = u < BP * WP;
        const int cg = (pb + HM - 1) * WM + pa + HM - 1;  // first point in the mu region
        const int cp = pb * WP + pa;                      // ... in the phi region
        const int cd = (pb + HR - 1) * WR + pa + HR - 1;  // ... in the rho region
        const real *j = (const real *)jq;
        real *F = (real *)Fq;
        unsigned off[RC], own = 0;
#pragma unroll
        for (int i = 0; i < RC; ++i) {
            off[i] = has ? S * node(pa - 1, pb + i - 1) : kOOB;
            if (has && inside(pa - 1, pb + i - 1)) own |= 1u << i;
        }
        real pj[RC][3];
        auto issue = [&](int g, bool ok) {  // j of plane g
            const size_t base = pbase(g);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const __amdgpu_buffer_rsrc_t rj = plane_rsrc(j + c * N + base, ok ? pbytesr : 0u);
#pragma unroll
                for (int i = 0; i < RC; ++i) bload(pj[i][c], rj, off[i]);
            }
        };
        double Aa[RC], Ab[RC], Ba[RC], Bb[RC], Ca[RC], Cb[RC], mc[RC];
#pragma unroll
        for (int i = 0; i < RC; ++i) Aa[i] = Ab[i] = Ba[i] = Bb[i] = Ca[i] = Cb[i] = mc[i] = 0.0;
        int g = wrap(tb - 4, kp.nz);
        issue(g, false);
        int s4 = 4;  // slot of plane t - 4; plane zs - 3 is in slot 0
        __syncthreads();
        for (int t = tb; t <= te; ++t) {
            const int p3 = t - 3, p = t - 4;
            const size_t base = pbase(g);
            real f[RC][3];
#pragma unroll
            for (int i = 0; i < RC; ++i) f[i][0] = f[i][1] = f[i][2] = (real)0;
            if (p3 >= zs - 2 && p3 <= ze + 1 && has) {
                double An[RC], Bn[RC], Cn[RC], mid[RC];
                grad_rows<WM, RC>(sm[p3 & 1], cg, An, Bn, Cn, mid);
                if (solid(g)) {
#pragma unroll
                    for (int i = 0; i < RC; ++i)
#pragma unroll
                        for (int c = 0; c < 3; ++c) sp[p & 1][c][cp + i * WP] = (real)0;
                } else if (p >= zs - 1) {
#pragma unroll
                    for (int i = 0; i < RC; ++i) {
                        real ph[3];
                        force_phi(Aa[i], Ab[i], An[i], Ba[i], Bb[i], Bn[i], Ca[i], Cn[i], sr[s4][cd + i * WR], mc[i], pj[i],
                                  f[i][0], f[i][1], f[i][2], ph);
#pragma unroll
                        for (int c = 0; c < 3; ++c) sp[p & 1][c][cp + i * WP] = ph[c];
                    }
                }
#pragma unroll
                for (int i = 0; i < RC; ++i) {
                    Aa[i] = Ab[i], Ba[i] = Bb[i], Ca[i] = Cb[i];
                    Ab[i] = An[i], Bb[i] = Bn[i], Cb[i] = Cn[i];
                    mc[i] = mid[i];
                }
            }
            // the next plane's loads go ahead of this plane's stores, so that
            // waiting for them does not wait for the stores
            g = next(g);
            issue(g, p + 1 >= zs - 1 && p + 1 <= ze);
            const bool out = p >= zs && p < ze;
            const __amdgpu_buffer_rsrc_t r0 = plane_rsrc(F + base, pbytesr);
            const __amdgpu_buffer_rsrc_t r1 = plane_rsrc(F + N + base, pbytesr);
            const __amdgpu_buffer_rsrc_t r2 = plane_rsrc(F + 2 * N + base, pbytesr);
#pragma unroll
            for (int i = 0; i < RC; ++i) {
                const unsigned o = out && ((own >> i) & 1u) ? off[i] : kOOB;
                bstore(f[i][0], r0, o);
                bstore(f[i][1], r1, o);
                bstore(f[i][2], r2, o);
            }
            s4 = s4 == 4 ? 0 : s4 + 1;
            __syncthreads();
        }
    } else if (wave >= 8 && wave < 8 + VD) {
        // ---- Q(t-6) from the in-plane parts of phi(t-7 .. t-5)
        const int u = (wave - 8) * 64 + lane, qa = u % TX, qb = u / TX * RD;
        const int cq = (qb + 1) * WP + qa + 1;  // first point in the phi region
        real *Q = (real *)Qq;
        unsigned off[RD];
#pragma unroll
        for (int i = 0; i < RD; ++i) off[i] = inside(qa, qb + i) ? S * node(qa, qb + i) : kOOB;
        real Xa[RD], Xb[RD], Ya[RD], Yb[RD], Za[RD], Zb[RD];
#pragma unroll
        for (int i = 0; i < RD; ++i) Xa[i] = Xb[i] = Ya[i] = Yb[i] = Za[i] = Zb[i] = (real)0;
        int g = wrap(tb - 6, kp.nz);
        __syncthreads();
        for (int t = tb; t <= te; ++t) {
            if (t - 5 >= zs - 1) {
                real Xn[RD], Yn[RD], Zn[RD];
                const int sl = (t - 5) & 1;
                div_rows<WP, RD>(sp[sl][0], sp[sl][1], sp[sl][2], cq, Xn, Yn, Zn);
                const size_t base = pbase(g);
                const __amdgpu_buffer_rsrc_t r0 = plane_rsrc(Q + base, pbytesr);
                const __amdgpu_buffer_rsrc_t r1 = plane_rsrc(Q + N + base, pbytesr);
                const __amdgpu_buffer_rsrc_t r2 = plane_rsrc(Q + 2 * N + base, pbytesr);
#pragma unroll
                for (int i = 0; i < RD; ++i) {
                    real qx, qy, qz;
                    q_of(Xa[i], Xb[i], Xn[i], Ya[i], Yb[i], Yn[i], Za[i], Zn[i], qx, qy, qz);
                    const unsigned o = t - 6 >= zs ? off[i] : kOOB;
                    bstore(qx, r0, o);
                    bstore(qy, r1, o);
                    bstore(qz, r2, o);
                    Xa[i] = Xb[i], Ya[i] = Yb[i], Za[i] = Zb[i];
                    Xb[i] = Xn[i], Yb[i] = Yn[i], Zb[i] = Zn[i];
                }
            }
            g = next(g);
            __syncthreads();
        }
    } else {
        // ---- rho(t) into LDS; mu(t-2) from Wx Wy rho of planes t-3, t-2, t-1
        const int u = (wave == VC ? 0 : wave - 11) * 64 + lane, ma = u % WM, mb = u / WM * RB;
        const bool has = u < BM * WM;
        const int cr = (mb + 1) * WR + ma + 1;  // first point in the rho region
        const int cm = mb * WM + ma;            // ... in the mu region
        unsigned offr[MR], off[RB], own = 0;
#pragma unroll
        for (int m = 0; m < MR; ++m) {
            const int r = u + m * VB * 64;
            offr[m] = r < NR ? 8u * node(r % WR - HR, r / WR - HR) : kOOB;
        }
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            off[i] = has && mb + i < YM ? 8u * node(ma - HM, mb + i - HM) : kOOB;
            if (has && inside(ma - HM, mb + i - HM)) own |= 1u << i;
        }
        double pr[MR], m0[RB];
        auto issue_rho = [&](int g, bool ok) {
            const __amdgpu_buffer_rsrc_t r = plane_rsrc(rho + pbase(g), ok ? pbytes8 : 0u);
#pragma unroll
            for (int m = 0; m < MR; ++m) bload(pr[m], r, offr[m]);
        };
        auto issue_mu0 = [&](int g, bool ok) {
            const __amdgpu_buffer_rsrc_t r = plane_rsrc(mu0 + pbase(g), ok ? pbytes8 : 0u);
#pragma unroll
            for (int i = 0; i < RB; ++i) bload(m0[i], r, off[i]);
        };
        // planes zs - 3 .. zs - 1 at once, then Wx Wy rho of the first two
        double P0[RB], P1[RB], rc[RB];
        int gn = wrap(zs - 3, kp.nz), g2 = next(gn);
        {
            double pa[MR], pb[MR];
            issue_rho(gn, true);
#pragma unroll
            for (int m = 0; m < MR; ++m) pa[m] = pr[m];
            issue_rho(g2, true);
#pragma unroll
            for (int m = 0; m < MR; ++m) pb[m] = pr[m];
            gn = next(g2);
            issue_rho(gn, true);
#pragma unroll
            for (int m = 0; m < MR; ++m) {
                sr[0][u + m * VB * 64] = pa[m];
                sr[1][u + m * VB * 64] = pb[m];
                sr[2][u + m * VB * 64] = pr[m];
            }
            gn = next(gn);
            issue_rho(gn, true);
            if (!MU0) issue_mu0(g2, true);
            __syncthreads();
            smooth_rows<WR, RB>(sr[0], cr, P0, rc);
            smooth_rows<WR, RB>(sr[1], cr, P1, rc);
        }
        int s0 = 3;  // slot of plane t
        for (int t = tb; t <= te; ++t) {
#pragma unroll
            for (int m = 0; m < MR; ++m)
                sr[s0][u + m * VB * 64] = pr[m];
            gn = next(gn);
            issue_rho(gn, t + 1 <= ze + 2);
            const int p = t - 2;
            double v[RB];
#pragma unroll
            for (int i = 0; i < RB; ++i) v[i] = 0.0;
            if (p <= ze + 1 && has) {
                double P2[RB], mid[RB];
                smooth_rows<WR, RB>(sr[s0 == 0 ? 4 : s0 - 1], cr, P2, mid);
                // (the mu0 of a solid plane is its mu, from k_wall_planes, whatever
                // the planes beside it hold)
                const double kap6 = kp.kappa * 6.0;
                const bool sol = solid(g2);
#pragma unroll
                for (int i = 0; i < RB; ++i) {
                    const double s27 = A1 * P0[i] + A0 * P1[i] + A1 * P2[i];
                    const double d = s27 - rc[i];
                    v[i] = (MU0 ? mu_bulk(kp, rc[i]) : m0[i]) - kap6 * (WALLS && sol ? 0.0 : d);
                    P0[i] = P1[i];
                    P1[i] = P2[i];
                    rc[i] = mid[i];
                }
#pragma unroll
                for (int i = 0; i < RB; ++i) sm[p & 1][cm + i * WM] = v[i];
            }
            const bool out = p >= zs && p < ze;
            const __amdgpu_buffer_rsrc_t rmu = plane_rsrc(mu + pbase(g2), pbytes8);
            g2 = next(g2);
            if (!MU0) issue_mu0(g2, p + 1 <= ze + 1);
#pragma unroll
            for (int i = 0; i < RB; ++i) bstore(v[i], rmu, out && ((own >> i) & 1u) ? off[i] : kOOB);
            s0 = s0 == 4 ? 0 : s0 + 1;
            __syncthreads();
        }
    }
}

// ---------------------------------------------------------------------------
// The solid planes of the march between walls: their density (Eqs. (37)-(38))
// and mu, the average of mu over the nine nodes beside each (Eq. (36)), which
// are formed here as the chain forms them.  mu goes to mu0's solid planes too:
// the march takes it from there like any mu0, so its loop has no branch for
// the walls (with a pointer or value chosen per plane it ran twice as long).
// One workgroup per 32 x 8 nodes of a plane.
// ---------------------------------------------------------------------------
constexpr int WTX = 32, WTY = 8, WNT = WTX * WTY;
__global__ __launch_bounds__(WNT) void k_wall_planes(KP kp, double *rho, double *mu0, double *mu) {
    constexpr int W2 = WTX + 4, N2 = W2 * (WTY + 4), W1 = WTX + 2, N1 = W1 * (WTY + 2);  // rho, mu regions
    __shared__ double sr[3][N2], sm[N1];
    const int ntx = (kp.nx + WTX - 1) / WTX;
    const int x0 = (int)blockIdx.x % ntx * WTX, y0 = (int)blockIdx.x / ntx * WTY;
    const int ps = blockIdx.y ? kp.nz - 1 : 0, pf = blockIdx.y ? kp.nz - 2 : 1;
    const int tid = threadIdx.x;
    auto node = [&](int x, int y) { return (unsigned)wrap(y0 + y, kp.ny) * kp.nx + (unsigned)wrap(x0 + x, kp.nx); };
    for (int r = tid; r < N2; r += WNT) {
        const unsigned n = node(r % W2 - 2, r / W2 - 2);
#pragma unroll
        for (int z = 0; z < 3; ++z)
            if (const int p = pf - 1 + z; p != 0 && p != kp.nz - 1) sr[z][r] = rho[(size_t)p * kp.plane + n];
        const int y = (int)(n / (unsigned)kp.nx), x = (int)(n - (unsigned)y * kp.nx);
        sr[ps - pf + 1][r] = wall_rho(kp, rho, x, y, ps);
        if (kp.nz == 3) sr[pf - ps + 1][r] = wall_rho(kp, rho, x, y, 2 * pf - ps);
    }
    __syncthreads();
    for (int r = tid; r < N1; r += WNT) {
        const int c = (r / W1 + 1) * W2 + r % W1 + 1;
        const double P0 = smooth2<W2>(sr[0], c), P1 = smooth2<W2>(sr[1], c), P2 = smooth2<W2>(sr[2], c);
        const double r0 = sr[1][c];
        const double s27 = A1 * P0 + A0 * P1 + A1 * P2;
        sm[r] = mu0[(size_t)pf * kp.plane + node(r % W1 - 1, r / W1 - 1)] - kp.kappa * 6.0 * (s27 - r0);
    }
    __syncthreads();
    const int a = tid % WTX, b = tid / WTX;
    if (x0 + a < kp.nx && y0 + b < kp.ny) {
        const size_t n = (size_t)ps * kp.plane + (unsigned)(y0 + b) * kp.nx + x0 + a;
        rho[n] = sr[ps - pf + 1][(b + 2) * W2 + a + 2];
        mu0[n] = mu[n] = smooth2<W1>(sm, (b + 1) * W1 + a + 1);
    }
}

// ---------------------------------------------------------------------------
// The same chain for small grids: a workgroup owns a TX x TY x CZ block,
// loads the block's whole rho region (halo HR in the plane, 3 in z) at once
// and then runs the three stencils one after the other.  In each, a thread
// marches the columns it owns through all planes of the region in registers
// (the sums of the march, in the same order, so the same bits), so the block
// passes three barriers in all instead of three per plane, and its loads wait
// for memory once.  The region is recomputed by the neighbouring blocks
// (mu on 3.5 times the owned nodes at 16 x 8 x 4), which only pays while the
// march is set by latency: at 32^3 in FP64 the march takes 25.6 us (seven
// iterations of 3.7 us, half of its 64-wide tile empty), this kernel 6 us.
// ---------------------------------------------------------------------------
// With a storage form P the workgroup then collides its own nodes and
// push-streams them (k_collide's node, same code): F, mu and Q stay in LDS and
// registers.  Between walls it also forms the density of the solid planes from
// the fluid plane beside them (as k_wall_rho), and with moving walls applies
// their term to the node's reflected populations after storing them (as
// k_wall_move): two launches a step instead of five (us per step with the wall
// kernels apart / inside, moving walls: FP64 32^3 26.2 / 17.3, 101 x 67 x 53 77.0
// / 68.1; FP32 64^3 37.5 / 30.4; still walls: FP64 32^3 20.5 / 17.6, 64^3 48.8 /
// 46.1, but 80^3 81.3 / 83.3 before 96^3 139 / 136).
// ---------------------------------------------------------------------------
constexpr int kFields = -1;  // P: mu, F and Q to memory, no collision
template <int P, class real, bool WALLS, int TX, int TY, int CZ, int NT, bool NTL>
__global__ __launch_bounds__(NT) void k_chain_block(KP kp, const double *__restrict__ rho,
                                                    const double *__restrict__ mu0, const void *jq,
                                                    double *__restrict__ mu, void *Fq, void *Qq, const void *fin_q,
                                                    void *fout_q) {
    constexpr bool STEP = P != kFields;
    // mu one node wider next to walls: Eq. (36) averages it over x +- 1, y +- 1
    constexpr int HM = WALLS ? 3 : 2, HR = HM + 1;
    constexpr int WR = TX + 2 * HR, NR = WR * (TY + 2 * HR), ZR = CZ + 6;  // rho region
    constexpr int WM = TX + 2 * HM, NM = WM * (TY + 2 * HM), ZM = CZ + 4;  // mu region
    constexpr int WP = TX + 2, NP = WP * (TY + 2), ZP = CZ + 2;            // phi region
    constexpr int MR = (NR + NT - 1) / NT, MM = (NM + NT - 1) / NT, MP = (NP + NT - 1) / NT;
    static_assert(TX * TY <= NT, "one owned column per thread");
    __shared__ double sr[ZR][NR];
    __shared__ double sm[ZM][NM];
    __shared__ real sp[ZP][3][NP];
    __shared__ real sf[STEP ? CZ : 1][3][TX * TY];  // F of the owned nodes

    const int ntx = (kp.nx + TX - 1) / TX;
    const unsigned ntiles = gridDim.x, nb = gridDim.x * gridDim.y;
    const unsigned hw = blockIdx.y * gridDim.x + blockIdx.x;
    const unsigned q = nb >> 3, rem = nb & 7u, xcd = hw & 7u;
    const unsigned lid = xcd * q + (xcd < rem ? xcd : rem) + (hw >> 3);
    const int tile = (int)(lid % ntiles), chunk = (int)(lid / ntiles);
    const int x0 = (tile % ntx) * TX, y0 = (tile / ntx) * TY;
    const int zs = kp.z0 + chunk * CZ, ze = min(zs + CZ, kp.z1);
    const int tid = threadIdx.x;
    const size_t N = kp.N;
    const real *j = (const real *)jq;
    real *F = (real *)Fq;
    real *Q = (real *)Qq;
    auto fluid = [&](int p) { return WALLS ? (p >= 1 && p <= kp.nz - 2) : true; };
    // wrapped index of a region coordinate; points past the grid's halo stand
    // for its last halo point (nothing reads them)
    auto wrap1 = [&](int v, int n) {
        v = min(v, n + HR - 1);
        if (n < HR) return wrap(v, n);
        return v < 0 ? v + n : (v >= n ? v - n : v);
    };
    auto node = [&](int x, int y) { return (unsigned)wrap1(y, kp.ny) * kp.nx + (unsigned)wrap1(x, kp.nx); };
    // first node of planes zs - 3 .. zs + CZ + 2 (outside a walled box they
    // wrap to planes whose values are not used)
    size_t pb[ZR];
    {
        int g = wrap(zs - 3, kp.nz);
#pragma unroll
        for (int z = 0; z < ZR; ++z) {
            pb[z] = (size_t)g * kp.plane;
            g = g + 1 == kp.nz ? 0 : g + 1;
        }
    }

    // the node of this thread's q-th collision (owned column cc, plane zs + cz)
    constexpr int NN = TX * TY * CZ, RN = (NN + NT - 1) / NT;
    auto col_of = [&](int q, int &cc, int &cz) {
        const int i = tid + q * NT;
        cc = i % (TX * TY);
        cz = i / (TX * TY);
        return i < NN && x0 + cc % TX < kp.nx && y0 + cc / TX < kp.ny && zs + cz < ze;
    };
    // its populations (the first node's at once, with the block's other loads)
    real f[STEP ? 27 : 1];
    auto load_f = [&](int q) {
        if constexpr (STEP) {
            int cc, cz;
            const Pops<P, NTL> fin(fin_q, kp);
            if (col_of(q, cc, cz)) {
                const unsigned row = (unsigned)(zs + cz) * (unsigned)kp.ny + (unsigned)(y0 + cc / TX);
#pragma unroll
                for (int i = 0; i < 27; ++i) f[i] = fin.ld(i, row, (unsigned)(x0 + cc % TX));
            }
        }
    };

    // every load of the block, before the first barrier
    double m0[MM][ZM];
    real pj[MP][ZP][3];
    unsigned orr[MR], om[MM], op[MP];
#pragma unroll
    for (int m = 0; m < MR; ++m) {
        const int r = min(tid + m * NT, NR - 1);
        orr[m] = node(x0 + r % WR - HR, y0 + r / WR - HR);
    }
#pragma unroll
    for (int m = 0; m < MM; ++m) {
        const int r = min(tid + m * NT, NM - 1);
        om[m] = node(x0 + r % WM - HM, y0 + r / WM - HM);
    }
#pragma unroll
    for (int m = 0; m < MP; ++m) {
        const int r = min(tid + m * NT, NP - 1);
        op[m] = node(x0 + r % WP - 1, y0 + r / WP - 1);
    }
    {
        double pr[MR][ZR];
#pragma unroll
        for (int z = 0; z < ZR; ++z)
#pragma unroll
            for (int m = 0; m < MR; ++m) pr[m][z] = rho[pb[z] + orr[m]];
#pragma unroll
        for (int z = 0; z < ZM; ++z)
#pragma unroll
            for (int m = 0; m < MM; ++m) m0[m][z] = mu0[pb[z + 1] + om[m]];
#pragma unroll
        for (int z = 0; z < ZP; ++z)
#pragma unroll
            for (int m = 0; m < MP; ++m)
#pragma unroll
                for (int c = 0; c < 3; ++c) pj[m][z][c] = j[c * N + pb[z + 2] + op[m]];
        load_f(0);
#pragma unroll
        for (int z = 0; z < ZR; ++z)
#pragma unroll
            for (int m = 0; m < MR; ++m)
                if (tid + m * NT < NR) sr[z][tid + m * NT] = pr[m][z];
    }
    if constexpr (STEP && WALLS) {  // the density of the solid planes, as k_wall_rho forms it
        auto wall = [&](int ps) {
#pragma unroll
            for (int m = 0; m < MR; ++m) {
                const int r = tid + m * NT;
                if (r < NR)
                    sr[ps - (zs - 3)][r] =
                        wall_rho(kp, rho, wrap1(x0 + r % WR - HR, kp.nx), wrap1(y0 + r / WR - HR, kp.ny), ps);
            }
        };
        if (zs <= 3) wall(0);
        if (zs + CZ + 2 >= kp.nz - 1) wall(kp.nz - 1);
    }
    __syncthreads();

    // mu of planes zs - 2 .. zs + CZ + 1 (fluid ones)
#pragma unroll
    for (int m = 0; m < MM; ++m) {
        const int r = tid + m * NT;
        if (r >= NM) continue;
        const int a = r % WM, b = r / WM, c = (b + 1) * WR + a + 1;
        const bool own = a >= HM && b >= HM && a < TX + HM && b < TY + HM && x0 + a - HM < kp.nx && y0 + b - HM < kp.ny;
        double P0 = smooth2<WR>(sr[0], c), P1 = smooth2<WR>(sr[1], c);
#pragma unroll
        for (int z = 0; z < ZM; ++z) {
            const int p = zs - 2 + z;
            const double P2 = smooth2<WR>(sr[z + 2], c);
            const double r0 = sr[z + 1][c];
            const double s27 = A1 * P0 + A0 * P1 + A1 * P2;
            const double v = m0[m][z] - kp.kappa * 6.0 * (s27 - r0);
            if (fluid(p)) {
                sm[z][r] = v;
                if (!STEP && own && p >= zs && p < ze) mu[pb[z + 1] + om[m]] = v;
            }
            P0 = P1;
            P1 = P2;
        }
    }
    __syncthreads();
    if constexpr (WALLS) {  // the solid planes inside the region, Eq. (36)
        const bool lo = zs <= 2, hi = ze + 1 >= kp.nz - 1;
        auto wall_mu = [&](int ps, int pf, bool write_out) {
            const int zw = ps - (zs - 2), zf = pf - (zs - 2);
#pragma unroll
            for (int m = 0; m < MM; ++m) {
                const int r = tid + m * NT, a = r % WM, b = r / WM;
                if (r >= NM || a < 1 || a > WM - 2 || b < 1 || b > TY + 2 * HM - 2) continue;
                const double v = smooth2<WM>(sm[zf], r);
                sm[zw][r] = v;
                if (!STEP && write_out && a >= HM && b >= HM && a < TX + HM && b < TY + HM && x0 + a - HM < kp.nx &&
                    y0 + b - HM < kp.ny)
                    mu[(size_t)ps * kp.plane + om[m]] = v;
            }
        };
        if (lo) wall_mu(0, 1, zs == 1);
        if (hi) wall_mu(kp.nz - 1, kp.nz - 2, ze == kp.nz - 1);
        if (lo || hi) __syncthreads();
    }

    // F and phi of planes zs - 1 .. zs + CZ
#pragma unroll
    for (int m = 0; m < MP; ++m) {
        const int r = tid + m * NT;
        if (r >= NP) continue;
        const int a = r % WP, b = r / WP;
        const int c = (b + HM - 1) * WM + a + HM - 1, cr = (b + HR - 1) * WR + a + HR - 1;
        const bool own = a >= 1 && b >= 1 && a <= TX && b <= TY && x0 + a - 1 < kp.nx && y0 + b - 1 < kp.ny;
        double Aa, Ba, Ca, Ab, Bb, Cb, Ac, Bc, Cc;
        plane_grad<WM>(sm[0], c, Aa, Ba, Ca);
        plane_grad<WM>(sm[1], c, Ab, Bb, Cb);
#pragma unroll
        for (int z = 0; z < ZP; ++z) {
            const int p = zs - 1 + z;
            plane_grad<WM>(sm[z + 2], c, Ac, Bc, Cc);
            if (fluid(p)) {
                real Fx, Fy, Fz, ph[3];
                force_phi(Aa, Ab, Ac, Ba, Bb, Bc, Ca, Cc, sr[z + 2][cr], sm[z + 1][c], pj[m][z], Fx, Fy, Fz, ph);
                for (int k = 0; k < 3; ++k) sp[z][k][r] = ph[k];
                if (own && p >= zs && p < ze) {
                    if constexpr (STEP) {
                        const int cc = (b - 1) * TX + a - 1;
                        sf[p - zs][0][cc] = Fx;
                        sf[p - zs][1][cc] = Fy;
                        sf[p - zs][2][cc] = Fz;
                    } else {
                        const size_t n = pb[z + 2] + op[m];
                        F[n] = Fx;
                        F[N + n] = Fy;
                        F[2 * N + n] = Fz;
                    }
                }
            } else {
                for (int k = 0; k < 3; ++k) sp[z][k][r] = (real)0;
            }
            Aa = Ab, Ba = Bb, Ca = Cb;
            Ab = Ac, Bb = Bc, Cb = Cc;
        }
    }
    __syncthreads();

    if constexpr (STEP) {
        // Q, collision and push-stream of the owned nodes
        const Pops<P> fout(fout_q, kp);
#pragma unroll
        for (int q = 0; q < RN; ++q) {
            if (q) load_f(q);
            int cc, cz;
            if (!col_of(q, cc, cz)) continue;
            const int a = cc % TX, b = cc / TX, c = (b + 1) * WP + a + 1;
            real X[3], Y[3], Z[3], qx, qy, qz;
#pragma unroll
            for (int d = 0; d < 3; ++d)
                plane_div<WP>(sp[cz + d][0], sp[cz + d][1], sp[cz + d][2], c, X[d], Y[d], Z[d]);
            q_of(X[0], X[1], X[2], Y[0], Y[1], Y[2], Z[0], Z[2], qx, qy, qz);
            collide_node(kp, f, sm[cz + 2][(b + HM) * WM + a + HM], sf[cz][0][cc], sf[cz][1][cc], sf[cz][2][cc], qx, qy,
                         qz);
            const int z = zs + cz;
            const Nb nb(kp, x0 + a, y0 + b, z);
            const unsigned row = nb.row(0, 0), x = (unsigned)(x0 + a);
            const bool wall_lo = WALLS && z == 1, wall_hi = WALLS && z == kp.nz - 2;
#pragma unroll
            for (int i = 0; i < 27; ++i) {
                const int c3 = czi(i);
                if ((c3 < 0 && wall_lo) || (c3 > 0 && wall_hi))
                    fout.st(26 - i, row, x, f[i]);
                else
                    fout.st(i, nb.row(cyi(i), c3), nb.xo(cxi(i)), f[i]);
            }
            if (WALLS && kp.moving && (wall_lo || wall_hi))
                wall_move_node<P>(kp, fout, sr[cz + 3][(b + HR) * WR + a + HR], sm[cz + 2][(b + HM) * WM + a + HM], z,
                                  row, x);
        }
        return;
    }
    // Q of the owned columns
    const int a = tid % TX, b = tid / TX;
    if (tid < TX * TY && x0 + a < kp.nx && y0 + b < kp.ny) {
        const int c = (b + 1) * WP + a + 1;
        const size_t n0 = (size_t)(y0 + b) * kp.nx + (x0 + a);
        real Xa, Ya, Za, Xb, Yb, Zb, Xc, Yc, Zc;
        plane_div<WP>(sp[0][0], sp[0][1], sp[0][2], c, Xa, Ya, Za);
        plane_div<WP>(sp[1][0], sp[1][1], sp[1][2], c, Xb, Yb, Zb);
#pragma unroll
        for (int z = 0; z < CZ; ++z) {
            plane_div<WP>(sp[z + 2][0], sp[z + 2][1], sp[z + 2][2], c, Xc, Yc, Zc);
            const int p = zs + z;
            if (p < ze) {
                const size_t n = pb[z + 3] + n0;
                real qx, qy, qz;
                q_of(Xa, Xb, Xc, Ya, Yb, Yc, Za, Zc, qx, qy, qz);
                Q[n] = qx;
                Q[N + n] = qy;
                Q[2 * N + n] = qz;
            }
            Xa = Xb, Ya = Yb, Za = Zb;
            Xb = Xc, Yb = Yc, Zb = Zc;
        }
    }
}

}  // namespace

// Planes per workgroup.  One workgroup fits a CU (LDS), and every march
// starts with six pipeline-fill planes, so chunks of c planes cost the
// busiest CU ceil(workgroups / CUs) x (c + 6) plane iterations; the chunk
// length from 64 down to 1 that minimises it is taken (the longer on ties;
// with powers of two only, 160^3 ran 32-plane chunks on 150 CUs, 137 us in
// FP64 against 76 for 20-plane ones on 240).  (128-plane chunks, which the
// count favours at 512^3, measured slower.)
constexpr unsigned kCUs = 256;  // MI355X
static int chain_chunk(const KP &kp, unsigned tiles) {
    const int nzf = kp.z1 - kp.z0;
    auto iters = [&](int c) {
        const size_t wg = (size_t)tiles * ((nzf + c - 1) / c);
        return ((wg + kCUs - 1) / kCUs) * (size_t)(c + 6);
    };
    int cz = 64;
    for (int c = 63; c >= 1; --c)
        if (iters(c) < iters(cz)) cz = c;
    return cz;
}

// The block kernel takes grids below 2^19 fluid nodes, where a march waits for
// its fill planes (us per step, march against block, two-pass path, periodic:
// FP64 64^3 54.1 / 49.6, 80^3 90.0 / 86.7; FP32 64^3 36.4 / 32.3, 80^3 60.3 /
// 59.2); beyond, the blocks' recomputed region costs more (96^3 FP64 132.9 /
// 139.6, FP32 80.3 / 86.0; 128^3 291 / 328).  A chunk length that the caller
// forces and the block kernel does not have (it has 1, 2 and 4) goes to a march,
// and so does a grid so long that its chunks exceed a launch's y dimension.
constexpr unsigned kBlockNodes = 1u << 19;
constexpr int BX = 16, BY = 8;  // 32x8, 32x4 and 16x4 blocks: 0-12 % slower per step
constexpr int kMaxGridY = 65535;
static bool block_chunks_fit(const KP &kp, int cz) { return (kp.z1 - kp.z0 + cz - 1) / cz <= kMaxGridY; }
static bool chain_block_grid(const KP &kp) { return kp.nfluid < kBlockNodes && block_chunks_fit(kp, 4); }

static size_t block_tiles(const KP &kp) { return (size_t)((kp.nx + BX - 1) / BX) * ((kp.ny + BY - 1) / BY); }

// the fewest planes that leave one workgroup per CU, else 4 (32^3: 1, 2, 4
// planes take 16.9, 18.2, 22.1 us per FP64 step; 64^3: 50.8, 44.0, 40.4), but no
// more than the grid has (one plane of 700 x 700, chunks of 4 / 1: FP64 101 / 77,
// FP32 83 / 55)
static int block_chunk(const KP &kp) {
    const size_t tiles = block_tiles(kp), nzf = kp.z1 - kp.z0;
    return tiles * nzf <= kCUs || nzf == 1 ? 1 : (tiles * ((nzf + 1) / 2) <= kCUs || nzf == 2 ? 2 : 4);
}

int chain_chunk_for(const KP &kp) {
    if (kp.chain_cz > 0) return kp.chain_cz;
    if (chain_block_grid(kp)) return block_chunk(kp);
    const unsigned ntx = (kp.nx + TX - 1) / TX, nty = (kp.ny + TY - 1) / TY;
    return chain_chunk(kp, ntx * nty);
}

template <int P, class real, bool WALLS, int CZ>
static void go_block(hipStream_t s, const KP &kp, const Bufs &b, const void *fin, void *fout) {
    // 256 threads hold the 240 mu columns; next to walls, with 308, 512 are
    // faster where a block has work for them (us per step at 96^3 FP64 145
    // against 148 with 256 and 158 with 320; at 32^3 22.6 against 21.9).
    // Blocks that also collide: 512 for 4 planes of the narrow forms (80^3 FP32
    // 46.5 against 47.5, walls 49.5 / 52.1; 67 x 63 x 61 FP16 32.4 / 33.7, walls 35.7 /
    // 40.0; 64^3 periodic alone 28.2 / 27.3), but in FP64 the populations of 512
    // nodes leave one block per CU (80^3 85.9 against 72.8)
    constexpr int NT = CZ == 4 && (WALLS || (P != kFields && sizeof(real) == 4)) ? 512 : 256;
    // a step's lattice that the last-level cache does not hold: not in the FP16
    // forms, 105 MiB at most at their limit of nodes
    constexpr bool beyond = P == LBFE_FP64 || P == LBFE_FP32;
    const dim3 g(block_tiles(kp), (kp.z1 - kp.z0 + CZ - 1) / CZ);
    if (!beyond || kp.keep2)
        k_chain_block<P, real, WALLS, BX, BY, CZ, NT, false>
            <<<g, NT, 0, s>>>(kp, b.rho, b.mu0, b.j, b.mu, b.F, b.Q, fin, fout);
    else if constexpr (beyond)
        k_chain_block<P, real, WALLS, BX, BY, CZ, NT, true>
            <<<g, NT, 0, s>>>(kp, b.rho, b.mu0, b.j, b.mu, b.F, b.Q, fin, fout);
}
template <int P, class real>
static hipError_t go_block(hipStream_t s, const KP &kp, const Bufs &b, int cz, const void *fin, void *fout) {
    auto go = [&](auto walls) {
        constexpr bool W = decltype(walls)::value;
        switch (cz) {
            case 1: go_block<P, real, W, 1>(s, kp, b, fin, fout); break;
            case 2: go_block<P, real, W, 2>(s, kp, b, fin, fout); break;
            default: go_block<P, real, W, 4>(s, kp, b, fin, fout); break;
        }
    };
    if (kp.walls)
        go(std::true_type{});
    else
        go(std::false_type{});
    return hipGetLastError();
}

// Node slots that the blocks of a one-launch FP64 step work through: whole
// tiles and chunks, and once more a chunk for every solid plane that its region
// of three planes beyond it reaches, whose density it forms.
static size_t block_slots(const KP &kp, int cz) {
    const size_t chunks = (kp.z1 - kp.z0 + cz - 1) / cz, beside = min(chunks, (size_t)(2 / cz + 1));
    return block_tiles(kp) * BX * BY * cz * (chunks + (kp.walls ? 2 * beside : 0));
}

// Planes per block of the step that runs chain and collide-stream in one
// launch (0: two).  It saves a launch and the 7 fields between the two, and
// pays with latency that few resident blocks hide and with the slots of its
// last tiles and chunks.  FP64 gains to 1.5 x 2^20 slots (us per step, two launches /
// one: 32^3 19.6 / 16.7, 64^3 49.4 / 40.4, 101 x 67 x 53 77.6 / 70.1, 96^3 135 /
// 122, 112^3 199 / 193, but 116^3 262 / 273 and 512 x 512 x 5 189 / 245 on 1.8e6
// and 2.1e6 slots), between walls to 2^20 (still, moving: 80^3 89 / 84, 95 / 83;
// 88^3 119 / 116, 127 / 122; 96^3 139 / 136, 145 / 146; but 104^3 180 / 197, 187 /
// 201; 192 x 192 x 24 132 / 138, 141 / 157; 400 x 400 x 5 89 / 113, 102 / 128).  FP32
// gains to 2^19 nodes (32^3 16.6 / 14.0, 64^3 33.6 / 30.8, 80^3 53.2 / 46.9, walls
// 58.6 / 49.8, moving 67.6 / 51.0, 96^3 80.5 / 84.2), FP16 populations to 5 x 2^16
// (32^3 16.6 / 12.9, 64^3 31.4 / 27.6, 101 x 67 x 45 33.4 / 34.6, walls 40.9 / 37.3),
// both to 2^17 where a single plane lies beside both walls (FP32 300 x 200 21.3 /
// 18.6, 400 x 300 28.0 / 28.8, 700 x 700 77 / 83, moving 101 / 124; FP16 moving 450 x
// 450 53 / 62).
// Between walls FP64 blocks of 4 planes take the LDS of one block per CU: 2
// planes (80^3 83 against 88).
int step_block_chunk(const KP &kp, int prec) {
    if (kp.masked) return 0;
    const int given = kp.chain_cz;
    if (given > 0 && given != 1 && given != 2 && given != 4) return 0;
    const int cz = given > 0 ? given : min(block_chunk(kp), kp.walls && prec == LBFE_FP64 ? 2 : 4);
    const bool small = prec == LBFE_FP64 ? block_slots(kp, cz) < (kp.walls ? 1u << 20 : 3u << 19)
                       : kp.nfluid < (kp.walls && kp.z1 - kp.z0 == 1 ? 1u << 17
                                      : prec == LBFE_FP32            ? 1u << 19
                                                                     : 5u << 16);
    return small && block_chunks_fit(kp, cz) ? cz : 0;
}

hipError_t launch_step_block(hipStream_t s, int prec, const KP &kp, const Bufs &b, int cur) {
    const void *fin = b.f[cur];
    void *fout = b.f[1 - cur];
    switch (prec) {
        case LBFE_FP64: return go_block<LBFE_FP64, double>(s, kp, b, kp.step_block, fin, fout);
        case LBFE_FP32: return go_block<LBFE_FP32, float>(s, kp, b, kp.step_block, fin, fout);
        case LBFE_FP16_DEV: return go_block<LBFE_FP16_DEV, float>(s, kp, b, kp.step_block, fin, fout);
        default: return go_block<LBFE_FP16_DEV_F0FP32, float>(s, kp, b, kp.step_block, fin, fout);
    }
}

static bool chain_is_block(const KP &kp, int cz) {
    return chain_block_grid(kp) && (cz == 1 || cz == 2 || cz == 4) && block_chunks_fit(kp, cz);
}

bool chain_forms_walls(const KP &kp) { return kp.walls && !chain_is_block(kp, chain_chunk_for(kp)); }

hipError_t launch_chain(hipStream_t s, int prec, const KP &kp, const Bufs &b) {
    const unsigned ntx = (kp.nx + TX - 1) / TX, nty = (kp.ny + TY - 1) / TY;
    const int cz = chain_chunk_for(kp);
    const int nzf = kp.z1 - kp.z0;
    if (chain_is_block(kp, cz))
        return prec == LBFE_FP64 ? go_block<kFields, double>(s, kp, b, cz, nullptr, nullptr)
                                 : go_block<kFields, float>(s, kp, b, cz, nullptr, nullptr);
    const dim3 grid(ntx * nty, (nzf + cz - 1) / cz);
    auto go = [&](auto real) {
        using R = decltype(real);
        if (kp.walls) {
            const unsigned gw = ((kp.nx + WTX - 1) / WTX) * ((kp.ny + WTY - 1) / WTY);
            k_wall_planes<<<dim3(gw, 2), WNT, 0, s>>>(kp, b.rho, b.mu0, b.mu);
            k_chain_march<R, false, true><<<grid, NTC, 0, s>>>(kp, b.rho, b.mu0, b.j, b.mu, b.F, b.Q, cz);
        } else if (kp.mu0_in_chain)
            k_chain_march<R, true, false><<<grid, NTC, 0, s>>>(kp, b.rho, b.mu0, b.j, b.mu, b.F, b.Q, cz);
        else
            k_chain_march<R, false, false><<<grid, NTC, 0, s>>>(kp, b.rho, b.mu0, b.j, b.mu, b.F, b.Q, cz);
    };
    if (prec == LBFE_FP64)
        go(double{});
    else
        go(float{});
    return hipGetLastError();
}

}  // namespace lbfe
