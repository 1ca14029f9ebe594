// Image-grid pass for small levels: 3D tiles of 4 x 4 x 16 voxels, one thread
// for every position a tile's stencils read.  Same arithmetic and output
// layout as the other image passes (P and the warp with float64 coordinates,
// the NGF term of Eq. 2 and its adjoint, the tile-local part of P^T, Eq. 3).
//
// A small level is bound by the length of its chain of dependent steps, not
// by its arithmetic: 32^3 is 512 tiles, two a CU.  So nothing is looped: the
// 928 positions (256 voxels, the 288 faces of the one-voxel halo, the 288 of
// the two-voxel halo and the 96 edges between) each have a thread, which
// warps it once; the index maps are in closed form instead of tables; P is
// interpolated along x first, by the threads that load the nodes; and the
// four stages are separated by four barriers.  Per launch, against the form that
// walked the halo in five rounds of 256 threads (kernel trace): 32^3 14.2 -> 7.5
// us, 64 x 80 x 48 22.8 -> 15.5, 64^3 22.6 -> 15.8.
#include "ngf_internal.h"

#include <math.h>

namespace ngf {

namespace {

constexpr int CX = 4, CY = 4, CZ = 16;                   // tile
constexpr int HX = CX + 4, HY = CY + 4, HZ = CZ + 4;     // box with the two-voxel halo
constexpr int NBOX = HX * HY * HZ;
constexpr int NTILE = CX * CY * CZ;                      // 256
constexpr int NF = 2 * (CX * CY + CX * CZ + CY * CZ);    // 288 faces of a halo
constexpr int NPOS = NTILE + 2 * NF + 4 * (CX + CY + CZ);  // 928
constexpr int SVX = (CX + 2) * CY * CZ, SVY = CX * (CY + 2) * CZ, SVZ = CX * CY * (CZ + 2);

__device__ inline int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

template <int R, bool GRAD>
struct Cube {
    static constexpr int NT = GRAD ? 960 : 576;          // NPOS or NTILE + NF, in whole waves
    static constexpr int QY = CY / R + 3, QZ = CZ / R + 3;
    static constexpr int NQ = HX * QY * QZ * 3;          // x-interpolated nodes of the box
    static constexpr int BX = CX / R, BY = CY / R, BZ = CZ / R;
    static constexpr int PX = BX + 1, PY = BY + 1, PZ = BZ + 1;
};

// position s in the box: tile, faces at distance 1, at distance 2, edges
__device__ inline void cube_pos(int s, int& bx, int& by, int& bz) {
    if (s < NTILE) {
        bx = 2 + (s >> 6);
        by = 2 + ((s >> 4) & 3);
        bz = 2 + (s & 15);
        return;
    }
    s -= NTILE;
    const int e = s >= NF ? 1 : 0;  // one further out
    if (s < 2 * NF) {
        s -= e * NF;
        if (s < 128) {
            bx = (s & 64) ? CX + 2 + e : 1 - e;
            by = 2 + ((s >> 4) & 3);
            bz = 2 + (s & 15);
        } else if (s < 256) {
            bx = 2 + ((s >> 4) & 3);
            by = (s & 64) ? CY + 2 + e : 1 - e;
            bz = 2 + (s & 15);
        } else {
            bx = 2 + ((s >> 3) & 3);
            by = 2 + ((s >> 1) & 3);
            bz = (s & 1) ? CZ + 2 + e : 1 - e;
        }
        return;
    }
    s -= 2 * NF;
    if (s < 64) {  // along z
        bx = (s & 16) ? CX + 2 : 1;
        by = (s & 32) ? CY + 2 : 1;
        bz = 2 + (s & 15);
    } else if (s < 80) {  // along y
        bx = (s & 1) ? CX + 2 : 1;
        by = 2 + ((s >> 2) & 3);
        bz = (s & 2) ? CZ + 2 : 1;
    } else {  // along x
        bx = 2 + ((s >> 2) & 3);
        by = (s & 1) ? CY + 2 : 1;
        bz = (s & 2) ? CZ + 2 : 1;
    }
}

template <int R>
__device__ inline double w1_of(int i) {
    return static_cast<double>(static_cast<float>(2 * (i % R) + 1) * (0.5f / R));
}
// weight of voxel l of the tile for its node n along an axis: the hat function
template <int R>
__device__ inline float hat(int l, int n) {
    return fmaxf(0.0f, 1.0f - fabsf((static_cast<float>(l) + 0.5f) * (1.0f / R) -
                                    static_cast<float>(n)));
}

template <int CTRL>
__device__ inline float dpp(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}

template <int R, bool GRAD, bool POW2>
__device__ __forceinline__ void cube_body(const ImagePassArgs& a, int block) {
    using L = Cube<R, GRAD>;
    constexpr int NT = L::NT;
    __shared__ double sQ[L::NQ];
    __shared__ float sT[NBOX], sR[NBOX];
    __shared__ float sV[GRAD ? SVX + SVY + SVZ : 1];
    __shared__ float sG[GRAD ? 3 * NTILE : 1];
    __shared__ double red[4];

    const int t = threadIdx.x;
    const int tile = xcd_tile(block, a.ntx * a.nty * a.ntz);
    const int tz = tile % a.ntz, ty = (tile / a.ntz) % a.nty, tx = tile / (a.ntz * a.nty);
    const int x0 = tx * CX, y0 = ty * CY, z0 = tz * CZ;
    const int mx = a.mx, my = a.my, mz = a.mz;
    const int sx = my * mz;

    // ---- nodes of the box, interpolated along x; R at this thread's position
    const int nnod = a.nx * a.ny * a.nz;
    const int qy0 = max(y0 - 2, 0) / R, qz0 = max(z0 - 2, 0) / R;
    for (int i = t; i < L::NQ; i += NT) {
        const int c = i % 3, r = i / 3;
        const int z = r % L::QZ, y = (r / L::QZ) % L::QY, bx = r / (L::QZ * L::QY);
        const int gx = clampi(x0 - 2 + bx, 0, mx - 1);
        const int jy = min(qy0 + y, a.ny - 1), jz = min(qz0 + z, a.nz - 1);
        const float* p = a.y + c * nnod + ((gx / R) * a.ny + jy) * a.nz + jz;
        const double v0 = p[0], v1 = p[a.ny * a.nz];
        sQ[i] = fma(w1_of<R>(gx), v1 - v0, v0);
    }
    int bx, by, bz;
    cube_pos(min(t, (GRAD ? NPOS : NTILE + NF) - 1), bx, by, bz);
    // the position's voxel (clamped: the value of a ghost is its voxel's) and
    // the voxel's place in the box
    const int gx = clampi(x0 - 2 + bx, 0, mx - 1), gy = clampi(y0 - 2 + by, 0, my - 1),
              gz = clampi(z0 - 2 + bz, 0, mz - 1);
    const int box = (bx * HY + by) * HZ + bz;
    sR[box] = a.R[gx * sx + gy * mz + gz];
    __syncthreads();

    // ---- P and the warp ---------------------------------------------------
    float dT[3];
    {
        const double* Q = sQ + 3 * ((bx * L::QY + (gy / R - qy0)) * L::QZ + (gz / R - qz0));
        const double wy = w1_of<R>(gy), wz = w1_of<R>(gz);
        const double hh[3] = {a.hx, a.hy, a.hz}, ih[3] = {a.ihx, a.ihy, a.ihz};
        const float fih[3] = {a.fihx, a.fihy, a.fihz};
        const int mm[3] = {mx, my, mz};
        int i0[3];
        float f[3], s[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double lo = fma(wz, Q[c + 3] - Q[c], Q[c]);
            const double up = fma(wz, Q[3 * L::QZ + c + 3] - Q[3 * L::QZ + c], Q[3 * L::QZ + c]);
            const double yh = fma(wy, up - lo, lo);
            // continuous index y_hat / h - 1/2 (a power-of-two spacing has an
            // exact reciprocal, any other is divided), clamped into the domain
            const double xi = POW2 ? fma(yh, ih[c], -0.5) : yh / hh[c] - 0.5;
            const double xc = fmin(fmax(xi, 0.0), static_cast<double>(mm[c] - 1));
            s[c] = xc == xi ? fih[c] : 0.0f;
            i0[c] = min(static_cast<int>(xc), mm[c] - 2);
            f[c] = static_cast<float>(xc - static_cast<double>(i0[c]));
        }
        const float* p = a.T + (i0[0] * sx + i0[1] * mz + i0[2]);
        const float v000 = p[0], v001 = p[1], v010 = p[mz], v011 = p[mz + 1];
        const float v100 = p[sx], v101 = p[sx + 1], v110 = p[sx + mz], v111 = p[sx + mz + 1];
        const float qx = 1.0f - f[0], qy = 1.0f - f[1], qz = 1.0f - f[2];
        const float c00 = fmaf(f[2], v001, qz * v000), c01 = fmaf(f[2], v011, qz * v010);
        const float c10 = fmaf(f[2], v101, qz * v100), c11 = fmaf(f[2], v111, qz * v110);
        const float c0 = fmaf(f[1], c01, qy * c00), c1 = fmaf(f[1], c11, qy * c10);
        sT[box] = fmaf(f[0], c1, qx * c0);
        if (GRAD) {
            const float d0 = c01 - c00, d1 = c11 - c10;
            const float e00 = v001 - v000, e01 = v011 - v010, e10 = v101 - v100, e11 = v111 - v110;
            dT[0] = (c1 - c0) * s[0];
            dT[1] = fmaf(f[0], d1, qx * d0) * s[1];
            const float ez0 = fmaf(f[1], e01, qy * e00), ez1 = fmaf(f[1], e11, qy * e10);
            dT[2] = fmaf(f[0], ez1, qx * ez0) * s[2];
        }
    }
    __syncthreads();

    // ---- NGF on the tile and the faces ------------------------------------
    const bool inside = x0 - 2 + bx < mx && y0 - 2 + by < my && z0 - 2 + bz < mz;
    if (t < (GRAD ? NTILE + NF : NTILE)) {
        const int p = ((gx - x0 + 2) * HY + (gy - y0 + 2)) * HZ + (gz - z0 + 2);
        const float gTx = (sT[p + HY * HZ] - sT[p - HY * HZ]) * a.i2hx;
        const float gTy = (sT[p + HZ] - sT[p - HZ]) * a.i2hy;
        const float gTz = (sT[p + 1] - sT[p - 1]) * a.i2hz;
        const float gRx = (sR[p + HY * HZ] - sR[p - HY * HZ]) * a.i2hx;
        const float gRy = (sR[p + HZ] - sR[p - HZ]) * a.i2hy;
        const float gRz = (sR[p + 1] - sR[p - 1]) * a.i2hz;
        const float tau = a.tau, rho = a.rho;
        const float aa = fmaf(gTx, gTx, fmaf(gTy, gTy, fmaf(gTz, gTz, tau * tau)));
        const float bb = fmaf(gRx, gRx, fmaf(gRy, gRy, fmaf(gRz, gRz, rho * rho)));
        const float ab = fmaf(gTx, gRx, fmaf(gTy, gRy, fmaf(gTz, gRz, tau * rho)));
        const float iaa = __builtin_amdgcn_rcpf(aa), ibb = __builtin_amdgcn_rcpf(bb);
        if (t < NTILE) {
            // 1 - r^2 = (aa bb - ab^2) / (aa bb) with a = (grad T, tau), b = (grad R,
            // rho), products unfused: exactly 0 when a = b (aa = bb = ab bit for bit)
            float lag;
            {
#pragma clang fp contract(off)
                lag = aa * bb - ab * ab;
            }
            double d = inside ? static_cast<double>(lag * iaa * ibb) : 0.0;
            for (int o = 32; o > 0; o >>= 1) d += __shfl_down(d, o, 64);
            if ((t & 63) == 0) red[t >> 6] = d;
        }
        if (GRAD) {
            // v = -hbar ab/(aa^2 bb) (aa grad R - ab grad T), products unfused (exactly 0
            // when grad T = grad R)
            const float coef = -a.hbar * ab * (iaa * iaa) * ibb;
            float vx, vy, vz;
            {
#pragma clang fp contract(off)
                vx = coef * (aa * gRx - ab * gTx);
                vy = coef * (aa * gRy - ab * gTy);
                vz = coef * (aa * gRz - ab * gTz);
            }
            // mirrored ghosts of the adjoint stencils' end rows
            if (gx != x0 - 2 + bx) vx = -vx;
            if (gy != y0 - 2 + by) vy = -vy;
            if (gz != z0 - 2 + bz) vz = -vz;
            const int lx = bx - 2, ly = by - 2, lz = bz - 2;
            const bool ix = lx >= 0 && lx < CX, iy = ly >= 0 && ly < CY, iz = lz >= 0 && lz < CZ;
            if (iy && iz) sV[((lx + 1) * CY + ly) * CZ + lz] = vx;
            if (ix && iz) sV[SVX + (lx * (CY + 2) + ly + 1) * CZ + lz] = vy;
            if (ix && iy) sV[SVX + SVY + (lx * CY + ly) * (CZ + 2) + lz + 1] = vz;
        }
    }
    __syncthreads();
    if (t == 0) a.dpart[tile] = (red[0] + red[1]) + (red[2] + red[3]);
    if (!GRAD) return;

    // ---- adjoint, and P^T along z over neighbouring lanes -------------------
    if (t < NTILE) {
        const int lx = bx - 2, ly = by - 2, lz = bz - 2;
        const float* Vx = sV + (lx * CY + ly) * CZ + lz;
        const float* Vy = sV + SVX + (lx * (CY + 2) + ly) * CZ + lz;
        const float* Vz = sV + SVX + SVY + (lx * CY + ly) * (CZ + 2) + lz;
        const float ex = Vx[0] - Vx[2 * CY * CZ], ey = Vy[0] - Vy[2 * CZ], ez = Vz[0] - Vz[2];
        const float e = inside ? fmaf(ex, a.i2hx, fmaf(ey, a.i2hy, ez * a.i2hz)) : 0.0f;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float g = e * dT[c];
            float v;
            if constexpr (R == 2) {
                // even lane: its cell's lower node, odd lane: the upper one
                v = fmaf(0.25f, dpp<0xB1>(g), 0.75f * g);
            } else {
                const float w1 = static_cast<float>(2 * (t & 3) + 1) * 0.125f;
                float lo = (1.0f - w1) * g, up = w1 * g;
                lo += dpp<0xB1>(lo);
                lo += dpp<0x4E>(lo);
                up += dpp<0xB1>(up);
                up += dpp<0x4E>(up);
                v = (t & 1) ? up : lo;
            }
            sG[c * NTILE + t] = v;
        }
    }
    __syncthreads();

    // ---- P^T along x and y: four threads a node, one for each row ------------
    float* out = a.part + static_cast<int64_t>(tile) * 3 * L::PX * L::PY * L::PZ;
    for (int i = t; i < 4 * 3 * L::PX * L::PY * L::PZ; i += NT) {
        const int q = i & 3, o = i >> 2;
        const int nz = o % L::PZ, ny = (o / L::PZ) % L::PY;
        const int nx = (o / (L::PZ * L::PY)) % L::PX, c = o / (L::PZ * L::PY * L::PX);
        const float* g = sG + c * NTILE + q * CZ;
        const int oa = min(nz, L::BZ - 1) * R, ob = max(nz - 1, 0) * R + 1;
        float v = 0.0f;
#pragma unroll
        for (int x = 0; x < CX; ++x) {
            const float va = nz < L::BZ ? g[x * CY * CZ + oa] : 0.0f;
            const float vb = nz > 0 ? g[x * CY * CZ + ob] : 0.0f;
            v = fmaf(hat<R>(x, nx), va + vb, v);
        }
        v *= hat<R>(q, ny);
        v += dpp<0xB1>(v);
        v += dpp<0x4E>(v);
        if (q == 0) out[o] = v;
    }
}

template <int R, bool GRAD, bool POW2>
__global__ __launch_bounds__((Cube<R, GRAD>::NT), 4) void k_image_cube(ImagePassArgs a) {
    if (a.gate && *a.gate == kOpNone) return;
    cube_body<R, GRAD, POW2>(a, blockIdx.x);
}

template <int R, bool POW2>
__global__ __launch_bounds__((Cube<R, true>::NT), 4) void k_image_cube_batch(
    const ImagePassArgs* args, const BlockRef* blk) {
    const BlockRef e = blk[blockIdx.x];
    const int pair = __builtin_amdgcn_readfirstlane(e.pair);  // uniform: scalar loads
    if (pair < 0) return;
    const ImagePassArgs a = args[pair];
    if (a.gate && *a.gate == kOpNone) return;
    cube_body<R, true, POW2>(a, __builtin_amdgcn_readfirstlane(e.block));
}

template <int R>
void launch_t(const ImagePassArgs& a, hipStream_t s) {
    const dim3 g(a.ntx * a.nty * a.ntz);
    if (a.want_grad) {
        if (a.pow2h)
            hipLaunchKernelGGL((k_image_cube<R, true, true>), g, dim3(Cube<R, true>::NT), 0, s, a);
        else
            hipLaunchKernelGGL((k_image_cube<R, true, false>), g, dim3(Cube<R, true>::NT), 0, s, a);
    } else {
        if (a.pow2h)
            hipLaunchKernelGGL((k_image_cube<R, false, true>), g, dim3(Cube<R, false>::NT), 0, s, a);
        else
            hipLaunchKernelGGL((k_image_cube<R, false, false>), g, dim3(Cube<R, false>::NT), 0, s,
                               a);
    }
}

template <int R>
void launch_batch_t(const ImagePassArgs* args, const BlockRef* blk, int nblk, bool pow2,
                    hipStream_t s) {
    if (pow2)
        hipLaunchKernelGGL((k_image_cube_batch<R, true>), dim3(nblk), dim3(Cube<R, true>::NT), 0,
                           s, args, blk);
    else
        hipLaunchKernelGGL((k_image_cube_batch<R, false>), dim3(nblk), dim3(Cube<R, true>::NT), 0,
                           s, args, blk);
}

}  // namespace

void launch_image_cube(const ImagePassArgs& a, int ratio, hipStream_t s) {
    if (ratio == 2)
        launch_t<2>(a, s);
    else if (ratio == 4)
        launch_t<4>(a, s);
}

// gradient form only (the batched rounds always want the gradient)
void launch_image_cube_batch(const ImagePassArgs* args, const BlockRef* blk, int nblk, int ratio,
                             bool pow2, hipStream_t s) {
    if (nblk <= 0) return;
    if (ratio == 2)
        launch_batch_t<2>(args, blk, nblk, pow2, s);
    else if (ratio == 4)
        launch_batch_t<4>(args, blk, nblk, pow2, s);
}

}  // namespace ngf
