// Node pass: completes the P^T gather of Eq. 3 (the at most eight image-tile
// partial sums of a node, in a fixed order), adds alpha grad S with grad S =
// hbar^y A(A(y - X)) and writes grad J once; block partials of S, max |grad J|
// and |grad J|^2.
//
// Up to a million nodes (kNodeForm): one workgroup per 3D tile of TX x TY x TZ
// nodes and all three components:
//   u = y - X on the tile and a two-node halo    -> LDS
//   A u on the tile and a one-node halo          -> LDS
//   A(A u), the partial sums and the gradient at the tile's nodes
// Ghost nodes replicate the boundary node, for u and for A u: a position
// outside the grid takes the value of the node clamped into it.
//
// The work is small there and the chain of dependent steps is what costs, so
// there are two barriers in all, a node's place in the partial sums is looked
// up once for its three components, from per-axis tables made once a
// workgroup, and the halo that the tiles share is read from the caches.  Node
// counts are mostly a power of two plus one: tiles of 17 along z (and 7 or 4
// along y) leave few idle threads there.
//
// Above that LDS traffic and the halo's work bound the tiles, and a workgroup
// marches along x instead, with the x neighbours in registers
// (node_march_body); the partial sums, 40 % of its traffic, bound it.
//
// Per launch, us (kernel trace), with the marching form at every size and one
// component a workgroup, and now: 17^3 nodes 11.0 and 7.1, 33^3 12.3 and 7.6,
// 64 x 68 x 53 15.5 and 14.2, 129^3 45.0 and 35.8.
#include "ngf_internal.h"

#include <math.h>

#include <atomic>
#include <type_traits>

namespace ngf {

namespace {

__device__ inline int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

__device__ inline double wave_sum(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    return v;
}
__device__ inline double wave_max(double v) {
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_down(v, o, 64));
    return v;
}

// Sums over the workgroup, written as the block's partials.
template <int NT, bool GRAD>
__device__ inline void node_sums(const NodePassArgs& a, int bid, double ssum, double gmax,
                                 double g2, double (*red)[NT / 64]) {
    ssum = wave_sum(ssum);
    if (GRAD) {
        gmax = wave_max(gmax);
        g2 = wave_sum(g2);
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[0][w] = ssum;
        red[1][w] = gmax;
        red[2][w] = g2;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0, m = 0.0, q = 0.0;
        for (int i = 0; i < NT / 64; ++i) {
            s += red[0][i];
            m = fmax(m, red[1][i]);
            q += red[2][i];
        }
        a.spart[bid] = s;
        if (GRAD) {
            a.gpart[2 * bid] = m;
            a.gpart[2 * bid + 1] = q;
        }
    }
}

__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const float* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, bytes, 0x00020000);
}
__device__ inline float bload(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}

// A stage over a box of PX planes along x, each of PY x PZ positions: the
// workgroup is split into groups of whole waves, one position of the plane a
// thread; group g takes planes g, g + groups, ...  So a thread's place in
// the plane is worked out once, and the plane is uniform over a wave.
template <int PX_, int PY_, int PZ_, int NT>
struct Planes {
    static constexpr int PX = PX_, PY = PY_, PZ = PZ_, N = PX * PY * PZ;
    static constexpr int W = (PY * PZ + 63) / 64 * 64, GROUPS = NT / W;
    static_assert(GROUPS >= 1, "a plane within the workgroup");
    int group, y, z;
    bool on;  // this thread has a position
    __device__ Planes(int t) {
        group = __builtin_amdgcn_readfirstlane(t / W);
        const int r = t - group * W;
        y = r / PZ;
        z = r - y * PZ;
        on = r < PY * PZ && group < GROUPS;
    }
};

// The three components of a vector field on the nodes, a descriptor each (a
// component is below 2^32 bytes, all three together need not be).
struct Comps {
    __amdgpu_buffer_rsrc_t r[3];
    __device__ Comps(const float* p, int nx, int ny, int nz) {
        const int64_t nn = static_cast<int64_t>(nx) * ny * nz;
#pragma unroll
        for (int c = 0; c < 3; ++c) r[c] = make_rsrc(p + c * nn, static_cast<uint32_t>(nn) * 4u);
    }
};

// GRAD: the gradient is wanted; GATHER: it collects the image-tile partials
// (else grad holds grad D on entry)
template <int TX, int TY, int TZ, int NT, bool GRAD, bool GATHER>
__device__ __forceinline__ void node_body(const NodePassArgs& a, int block) {
    using U = Planes<TX + 4, TY + 4, TZ + 4, NT>;
    using A = Planes<TX + 2, TY + 2, TZ + 2, NT>;
    using N = Planes<TX, TY, TZ, NT>;
    __shared__ float su[3 * U::N];
    __shared__ float sA[3 * A::N];
    __shared__ int4 stab[GATHER ? TX + TY + TZ : 1];
    __shared__ double red[3][NT / 64];

    const int t = threadIdx.x;
    const int bid = xcd_tile(block, a.nbx * a.nby * a.nbz);
    const int bz = bid % a.nbz, by = (bid / a.nbz) % a.nby, bx = bid / (a.nbz * a.nby);
    const int x0 = bx * TX, y0 = by * TY, z0 = bz * TZ;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int mx = a.mx, my = a.my, mz = a.mz, ex = a.tex, ey = a.tey, ez = a.tez;
    const uint32_t plane4 = static_cast<uint32_t>(ny * nz) * 4u;

    // u = y - X
    {
        const U u(t);
        if (u.on) {
            const Comps Y(a.y, nx, ny, nz);
            const int cy = clampi(y0 - 2 + u.y, 0, ny - 1), cz = clampi(z0 - 2 + u.z, 0, nz - 1);
            const uint32_t off = static_cast<uint32_t>(cy * nz + cz) * 4u;
            const double Xy = static_cast<double>(cy) * a.hyy, Xz = static_cast<double>(cz) * a.hyz;
            constexpr int K = (U::PX + U::GROUPS - 1) / U::GROUPS;
            float v[K][3];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int cx = clampi(x0 - 2 + u.group + k * U::GROUPS, 0, nx - 1);
                const uint32_t p = static_cast<uint32_t>(cx) * plane4;
#pragma unroll
                for (int c = 0; c < 3; ++c) v[k][c] = bload(Y.r[c], off, p);
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int ux = u.group + k * U::GROUPS;
                if (ux >= U::PX) break;
                const double Xx = static_cast<double>(clampi(x0 - 2 + ux, 0, nx - 1)) * a.hyx;
                float* o = su + (ux * U::PY + u.y) * U::PZ + u.z;
                o[0] = static_cast<float>(static_cast<double>(v[k][0]) - Xx);
                o[U::N] = static_cast<float>(static_cast<double>(v[k][1]) - Xy);
                o[2 * U::N] = static_cast<float>(static_cast<double>(v[k][2]) - Xz);
            }
        }
    }
    // image tiles that hold a node in their blocks, per axis
    if (GATHER && t >= NT - (TX + TY + TZ)) {
        const int i = t - (NT - (TX + TY + TZ));
        const bool ix = i < TX, iy = !ix && i < TX + TY;
        const int j = ix ? x0 + i : (iy ? y0 + i - TX : z0 + i - TX - TY);
        const int m = ix ? mx : (iy ? my : mz), n = ix ? nx : (iy ? ny : nz);
        const NodeTiles k = node_tiles(min(j, n - 1), m, n, ix ? ex : (iy ? ey : ez));
        stab[i] = make_int4(k.ta, k.la, k.tb, k.lb);
    }
    __syncthreads();
    // A u; a ghost's is that of the node clamped into the grid
    {
        const A p(t);
        if (p.on) {
            const int cy = clampi(y0 - 1 + p.y, 0, ny - 1), cz = clampi(z0 - 1 + p.z, 0, nz - 1);
            const int yz = (cy - y0 + 2) * U::PZ + (cz - z0 + 2);
            for (int ax = p.group; ax < A::PX; ax += A::GROUPS) {
                const int cx = clampi(x0 - 1 + ax, 0, nx - 1);
                const float* u = su + (cx - x0 + 2) * (U::PY * U::PZ) + yz;
                float* o = sA + (ax * A::PY + p.y) * A::PZ + p.z;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const float u0 = u[c * U::N];
                    const float lx = u[c * U::N + U::PY * U::PZ] - 2.0f * u0 +
                                     u[c * U::N - U::PY * U::PZ];
                    const float ly = u[c * U::N + U::PZ] - 2.0f * u0 + u[c * U::N - U::PZ];
                    const float lz = u[c * U::N + 1] - 2.0f * u0 + u[c * U::N - 1];
                    o[c * A::N] = fmaf(lx, a.ihy2x, fmaf(ly, a.ihy2y, lz * a.ihy2z));
                }
            }
        }
    }
    __syncthreads();
    double ssum = 0.0, gmax = 0.0, g2 = 0.0;
    const N n(t);
    if (n.on && y0 + n.y < ny && z0 + n.z < nz) {
        const float sc = a.gscale != nullptr ? static_cast<float>(*a.gscale) : 1.0f;
        const int NP = a.px * a.py * a.pz, PYZ = a.py * a.pz;
        const int64_t xslab = static_cast<int64_t>(a.nty) * a.ntz * 3 * NP;
        const int64_t nn = static_cast<int64_t>(nx) * ny * nz;
        // the node's (y, z) place in the blocks of its image tiles: j = 2 oy + oz,
        // the second tile along y if oy, along z if oz (negative: none)
        int yz[4] = {-1, -1, -1, -1};
        if (GRAD && GATHER) {
            const int4 ky = stab[TX + n.y], kz = stab[TX + TY + n.z];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int ttY = (j >> 1) ? ky.z : ky.x, ttZ = (j & 1) ? kz.z : kz.x;
                const int lY = (j >> 1) ? ky.w : ky.y, lZ = (j & 1) ? kz.w : kz.y;
                if (ttY >= 0 && ttZ >= 0) yz[j] = (ttY * a.ntz + ttZ) * 3 * NP + lY * a.pz + lZ;
            }
        }
        for (int x = n.group; x < TX && x0 + x < nx; x += N::GROUPS) {
            const int64_t k = (static_cast<int64_t>(x0 + x) * ny + (y0 + n.y)) * nz + (z0 + n.z);
            float gd[3] = {0.0f, 0.0f, 0.0f};
            if (GRAD && GATHER) {
                const int4 kx = stab[x];
#pragma unroll
                for (int o = 0; o < 2; ++o) {
                    const int ttx = __builtin_amdgcn_readfirstlane(o ? kx.z : kx.x);
                    if (ttx < 0) continue;
                    const float* p = a.part + ttx * xslab +
                                     __builtin_amdgcn_readfirstlane(o ? kx.w : kx.y) * PYZ;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (j > 0 && yz[j] < 0) continue;
                        gd[0] += p[yz[j]];
                        gd[1] += p[yz[j] + NP];
                        gd[2] += p[yz[j] + 2 * NP];
                    }
                }
            } else if (GRAD) {
#pragma unroll
                for (int c = 0; c < 3; ++c) gd[c] = a.grad[c * nn + k];
            }
            const float* q = sA + ((x + 1) * A::PY + (n.y + 1)) * A::PZ + (n.z + 1);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const float au = q[c * A::N];
                ssum += static_cast<double>(au) * static_cast<double>(au);
                if (GRAD) {
                    const float lx = q[c * A::N + A::PY * A::PZ] - 2.0f * au +
                                     q[c * A::N - A::PY * A::PZ];
                    const float ly = q[c * A::N + A::PZ] - 2.0f * au + q[c * A::N - A::PZ];
                    const float lz = q[c * A::N + 1] - 2.0f * au + q[c * A::N - 1];
                    const float aau = fmaf(lx, a.ihy2x, fmaf(ly, a.ihy2y, lz * a.ihy2z));
                    const float g = fmaf(a.alpha_hbary * sc, aau, GATHER ? sc * gd[c] : gd[c]);
                    a.grad[c * nn + k] = g;
                    gmax = fmax(gmax, static_cast<double>(fabsf(g)));
                    g2 += static_cast<double>(g) * static_cast<double>(g);
                }
            }
        }
    }
    node_sums<NT, GRAD>(a, bid, ssum, gmax, g2, red);
}

// Large grids.  A workgroup owns a tile of NY x NZ nodes in (y, z) and a chunk
// of planes along x and walks them, all three components together.  Thread t
// owns one node of every plane and one position of the in-plane halo (t <
// RING): its u and A u of three planes stay in its registers, LDS holds two
// planes of each for the neighbours in the plane.  Step k takes in plane pu,
// forms A u of plane pu - 1 and A(A u) and the gradient of plane pu - 2 from
// what earlier steps wrote to LDS, so one barrier a step suffices.
template <int NY, int NZ, int NT, bool GRAD, bool GATHER>
__device__ __forceinline__ void node_march_body(const NodePassArgs& a, int block) {
    constexpr int UZ = NZ + 4, NU = (NY + 4) * UZ;
    constexpr int AZ = NZ + 2, NA = (NY + 2) * AZ;
    constexpr int FACE = 2 * (NY + NZ), RING = 2 * FACE + 4;
    static_assert(NY * NZ <= NT && RING <= NT, "one node and one halo position a thread");
    __shared__ float su[2 * 3 * NU];
    __shared__ float sA[2 * 3 * NA];
    __shared__ int4 sxt[GATHER ? kNodeChunkMax : 1];
    __shared__ double red[3][NT / 64];

    const int t = threadIdx.x;
    const int bid = xcd_tile(block, a.nbx * a.nby * a.nbz);
    const int bz = bid % a.nbz, by = (bid / a.nbz) % a.nby, bx = bid / (a.nbz * a.nby);
    const int x0 = bx * a.cxn, y0 = by * NY, z0 = bz * NZ;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int xend = min(x0 + a.cxn, nx);
    const uint32_t plane4 = static_cast<uint32_t>(ny * nz) * 4u;
    const Comps Y(a.y, nx, ny, nz);
    const int64_t nn = static_cast<int64_t>(nx) * ny * nz;

    // the thread's node (A) and halo position (C), clamped into the grid: the
    // value of a ghost, of u and of A u, is its node's
    const int la = min(t, NY * NZ - 1);
    const int ly = la / NZ, lz = la - ly * NZ;
    const bool own = t < NY * NZ && y0 + ly < ny && z0 + lz < nz;
    const int cyA = min(y0 + ly, ny - 1), czA = min(z0 + lz, nz - 1);
    const int s = min(t, RING - 1);
    const int e = s >= FACE ? 1 : 0;  // one further out
    int byC, bzC;                     // in the box with the two-node halo
    {
        const int o = s - e * FACE;
        if (o < 2 * NZ) {
            byC = o < NZ ? 1 - e : NY + 2 + e;
            bzC = 2 + o % NZ;
        } else if (o < FACE) {
            const int q = o - 2 * NZ;
            byC = 2 + (q >> 1);
            bzC = (q & 1) ? NZ + 2 + e : 1 - e;
        } else {  // the corners of the one-node halo
            const int q = o - FACE;
            byC = (q & 1) ? NY + 2 : 1;
            bzC = (q & 2) ? NZ + 2 : 1;
        }
    }
    const bool ring = t < RING, face = t < FACE;
    const int cyC = clampi(y0 - 2 + byC, 0, ny - 1), czC = clampi(z0 - 2 + bzC, 0, nz - 1);
    const uint32_t offA = static_cast<uint32_t>(cyA * nz + czA) * 4u;
    const uint32_t offC = static_cast<uint32_t>(cyC * nz + czC) * 4u;
    const int boxA = (ly + 2) * UZ + lz + 2, ctrA = (cyA - y0 + 2) * UZ + (czA - z0 + 2);
    const int boxC = byC * UZ + bzC, ctrC = (cyC - y0 + 2) * UZ + (czC - z0 + 2);
    const int auA = (ly + 1) * AZ + lz + 1, auC = (byC - 1) * AZ + bzC - 1;
    const double XA[2] = {static_cast<double>(cyA) * a.hyy, static_cast<double>(czA) * a.hyz};
    const double XC[2] = {static_cast<double>(cyC) * a.hyy, static_cast<double>(czC) * a.hyz};
    const float sc = a.gscale != nullptr ? static_cast<float>(*a.gscale) : 1.0f;

    // places in the blocks of the image-tile partials: along x a table per
    // plane of the chunk, in (y, z) four offsets (j = 2 oy + oz: the second
    // tile along y if oy, along z if oz; negative: none)
    const int NP = a.px * a.py * a.pz, PYZ = a.py * a.pz;
    const int64_t xslab = static_cast<int64_t>(a.nty) * a.ntz * 3 * NP;
    int yz[4] = {-1, -1, -1, -1};
    if (GRAD && GATHER) {
        const NodeTiles ky = node_tiles(cyA, a.my, ny, a.tey), kz = node_tiles(czA, a.mz, nz, a.tez);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int tty = (j >> 1) ? ky.tb : ky.ta, ttz = (j & 1) ? kz.tb : kz.ta;
            const int lyy = (j >> 1) ? ky.lb : ky.la, lzz = (j & 1) ? kz.lb : kz.la;
            if (tty >= 0 && ttz >= 0) yz[j] = (tty * a.ntz + ttz) * 3 * NP + lyy * a.pz + lzz;
        }
        for (int i = t; i < xend - x0; i += NT) {
            const NodeTiles k = node_tiles(x0 + i, a.mx, nx, a.tex);
            sxt[i] = make_int4(k.ta, k.la, k.tb, k.lb);
        }
    }

    float vA[3], vC[3];  // y of the plane that enters next
    auto load_y = [&](int p) {
        const uint32_t o = static_cast<uint32_t>(clampi(p, 0, nx - 1)) * plane4;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            vA[c] = bload(Y.r[c], offA, o);
            vC[c] = bload(Y.r[c], offC, o);
        }
    };
    float uA[3][3] = {}, uC[3][3] = {}, aA[3][3] = {};  // [plane slot][component]
    double ssum = 0.0, gmax = 0.0, g2 = 0.0;
    load_y(x0 - 2);
    __syncthreads();  // sxt

    const int nstep = xend - x0 + 4;
    auto step = [&](auto slot, const int k) {
        constexpr int S = decltype(slot)::value;
        constexpr int S0 = S % 3, S1 = (S + 2) % 3, S2 = (S + 1) % 3;
        constexpr int P0 = S & 1, P1 = P0 ^ 1;  // LDS slots written in this step, in the last one
        const int pu = x0 - 2 + k;
        const int po = pu - 2;
        const bool out = po >= x0;
        // the first image tile's partial sums, in flight over the stencils
        float gd[3] = {0.0f, 0.0f, 0.0f}, gz[3] = {0.0f, 0.0f, 0.0f};
        int tta = 0, ttb = -1, lxa = 0, lxb = 0;
        const float* part = a.part;
        if (GRAD && GATHER && out) {
            const int4 xt = sxt[po - x0];
            tta = __builtin_amdgcn_readfirstlane(xt.x);
            lxa = __builtin_amdgcn_readfirstlane(xt.y);
            ttb = __builtin_amdgcn_readfirstlane(xt.z);
            lxb = __builtin_amdgcn_readfirstlane(xt.w);
            part += tta * xslab + lxa * PYZ;
#pragma unroll
            for (int c = 0; c < 3; ++c) gd[c] = part[yz[0] + c * NP];
            if (yz[1] >= 0) {
#pragma unroll
                for (int c = 0; c < 3; ++c) gz[c] = part[yz[1] + c * NP];
            }
        }
        // u of plane pu
        const double Xx = static_cast<double>(clampi(pu, 0, nx - 1)) * a.hyx;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            uA[S0][c] = static_cast<float>(static_cast<double>(vA[c]) - (c == 0 ? Xx : XA[c - 1]));
            uC[S0][c] = static_cast<float>(static_cast<double>(vC[c]) - (c == 0 ? Xx : XC[c - 1]));
        }
        if (k + 1 < nstep) load_y(pu + 1);
        // A u of plane pu - 1
        auto lap = [&](float um, float u0, float up, float ym, float yp, float zm, float zp) {
            const float lx = up - 2.0f * u0 + um;
            const float lyv = yp - 2.0f * u0 + ym;
            const float lzv = zp - 2.0f * u0 + zm;
            return fmaf(lx, a.ihy2x, fmaf(lyv, a.ihy2y, lzv * a.ihy2z));
        };
        if (k >= 2) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const float* U = su + (P1 * 3 + c) * NU;
                float* A = sA + (P0 * 3 + c) * NA;
                aA[S0][c] = lap(uA[S2][c], uA[S1][c], uA[S0][c], U[ctrA - UZ], U[ctrA + UZ],
                                U[ctrA - 1], U[ctrA + 1]);
                if (t < NY * NZ) A[auA] = aA[S0][c];
                if (face)
                    A[auC] = lap(uC[S2][c], uC[S1][c], uC[S0][c], U[ctrC - UZ], U[ctrC + UZ],
                                 U[ctrC - 1], U[ctrC + 1]);
            }
        }
        // A(A u) and the gradient of plane pu - 2; across the grid's ends the
        // ghost plane of A u is the boundary plane's
        if (out && own) {
            const int64_t g0 = static_cast<int64_t>(po) * ny * nz + (offA >> 2);
            if (GRAD && !GATHER) {
#pragma unroll
                for (int c = 0; c < 3; ++c) gd[c] = a.grad[c * nn + g0];
            }
            if (GRAD && GATHER) {
                if (yz[1] >= 0) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) gd[c] += gz[c];
                }
                auto add = [&](const float* p, int o) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) gd[c] += p[o + c * NP];
                };
                if (yz[2] >= 0) {
                    add(part, yz[2]);
                    if (yz[3] >= 0) add(part, yz[3]);
                }
                if (ttb >= 0) {
                    const float* p = a.part + ttb * xslab + lxb * PYZ;
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (j == 0 || yz[j] >= 0) add(p, yz[j]);
                }
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const float* A = sA + (P1 * 3 + c) * NA + auA;
                const float au = aA[S1][c];
                ssum += static_cast<double>(au) * static_cast<double>(au);
                if (GRAD) {
                    const float aau = lap(po > 0 ? aA[S2][c] : au, au, po + 1 < nx ? aA[S0][c] : au,
                                          A[-AZ], A[AZ], A[-1], A[1]);
                    const float g = fmaf(a.alpha_hbary * sc, aau, GATHER ? sc * gd[c] : gd[c]);
                    a.grad[c * nn + g0] = g;
                    gmax = fmax(gmax, static_cast<double>(fabsf(g)));
                    g2 += static_cast<double>(g) * static_cast<double>(g);
                }
            }
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            float* U = su + (P0 * 3 + c) * NU;
            if (t < NY * NZ) U[boxA] = uA[S0][c];
            if (ring) U[boxC] = uC[S0][c];
        }
        __syncthreads();
    };
    for (int k = 0; k < nstep; k += 6) {
        step(std::integral_constant<int, 0>(), k);
        if (k + 1 >= nstep) break;
        step(std::integral_constant<int, 1>(), k + 1);
        if (k + 2 >= nstep) break;
        step(std::integral_constant<int, 2>(), k + 2);
        if (k + 3 >= nstep) break;
        step(std::integral_constant<int, 3>(), k + 3);
        if (k + 4 >= nstep) break;
        step(std::integral_constant<int, 4>(), k + 4);
        if (k + 5 >= nstep) break;
        step(std::integral_constant<int, 5>(), k + 5);
    }
    node_sums<NT, GRAD>(a, bid, ssum, gmax, g2, red);
}

template <int FORM, bool GRAD, bool GATHER>
__device__ __forceinline__ void node_form(const NodePassArgs& a, int block) {
    constexpr NodeForm F = kNodeForm[FORM];
    if constexpr (F.x > 0)
        node_body<F.x, F.y, F.z, F.threads, GRAD, GATHER>(a, block);
    else
        node_march_body<F.y, F.z, F.threads, GRAD, GATHER>(a, block);
}
template <int FORM, bool GRAD, bool GATHER>
__global__ __launch_bounds__((kNodeForm[FORM].threads), 4) void k_node_pass(NodePassArgs a) {
    if (a.gate && *a.gate == kOpNone) return;
    node_form<FORM, GRAD, GATHER>(a, blockIdx.x);
}

// the batched rounds always want the gradient gathered from the image pass
template <int FORM>
__global__ __launch_bounds__((kNodeForm[FORM].threads), 4) void k_node_pass_batch(
    const NodePassArgs* args, const BlockRef* blk) {
    const BlockRef e = blk[blockIdx.x];
    const int pair = __builtin_amdgcn_readfirstlane(e.pair);  // uniform: scalar loads
    if (pair < 0) return;
    const NodePassArgs a = args[pair];
    if (a.gate && *a.gate == kOpNone) return;
    node_form<FORM, true, true>(a, __builtin_amdgcn_readfirstlane(e.block));
}

template <int FORM>
void launch_form(const NodePassArgs& a, hipStream_t s) {
    const dim3 g(a.nbx * a.nby * a.nbz), b(kNodeForm[FORM].threads);
    if (!a.want_grad)
        hipLaunchKernelGGL((k_node_pass<FORM, false, false>), g, b, 0, s, a);
    else if (a.gather)
        hipLaunchKernelGGL((k_node_pass<FORM, true, true>), g, b, 0, s, a);
    else
        hipLaunchKernelGGL((k_node_pass<FORM, true, false>), g, b, 0, s, a);
}

}  // namespace

int node_march_slots() {
    static std::atomic<int> cache[16];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) dev = 0;
    std::atomic<int>& slot = cache[dev & 15];
    int v = slot.load();
    if (v > 0) return v;
    int per_cu = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_node_pass<2, true, true>,
                                                     kNodeForm[2].threads, 0) != hipSuccess ||
        per_cu < 1)
        per_cu = 2;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus < 1)
        cus = 256;
    (void)hipGetLastError();
    v = per_cu * cus;
    slot.store(v);
    return v;
}

void launch_node_pass(const NodePassArgs& a, hipStream_t s) {
    if (a.form == 0)
        launch_form<0>(a, s);
    else if (a.form == 1)
        launch_form<1>(a, s);
    else
        launch_form<2>(a, s);
}

void launch_node_pass_batch(const NodePassArgs* args, const BlockRef* blk, int nblk, int form,
                            hipStream_t s) {
    if (nblk <= 0) return;
    const dim3 g(nblk), b(kNodeForm[form].threads);
    if (form == 0)
        hipLaunchKernelGGL(k_node_pass_batch<0>, g, b, 0, s, args, blk);
    else if (form == 1)
        hipLaunchKernelGGL(k_node_pass_batch<1>, g, b, 0, s, args, blk);
    else
        hipLaunchKernelGGL(k_node_pass_batch<2>, g, b, 0, s, args, blk);
}

}  // namespace ngf
