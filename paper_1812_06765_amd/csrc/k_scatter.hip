// Template gradient of the differentiation form: dD/dT[k] = sum_i e_i W(i -> k),
// the transpose of the trilinear warp, from the sensitivities e of the image
// pass (which stores them, see ImagePassArgs::sens).
//
// A scatter of eight weighted values a voxel.  Sent to memory one by one, the
// atomics are what it costs (8 a voxel, most of them in lines that the
// neighbours' go to as well).  A workgroup therefore takes a tile of
// SX x SY x SZ voxels, finds the box of template cells that they reach, adds
// them up in LDS, and sends each box entry once: about two atomics a voxel for a
// smooth deformation.  The LDS sums are float64 for their rate: a ds_add_f64 of
// a wave takes 10 cycles, a ds_add_f32 three a lane.  A box larger than kScatterBox entries (a strongly
// expanding or torn deformation) goes to memory directly.
// A thread owns a (y, z) column of the tile and walks its SX planes, with y
// interpolated in its column at the two node planes around x in registers, as
// the standalone P does.  Its cells, fractions and sensitivities fill the 128
// registers of two workgroups a CU and 5 to 7 more, which spill.
// 128^3: 29 us, and 37 for the image pass that stores e, against 229 us for the
// 3D-tile image pass that sends eight atomics a voxel to memory (102 us here
// with float32 sums in LDS).
#include "ngf_internal.h"

#include <math.h>

#include <type_traits>

namespace ngf {

namespace {

constexpr int SX = 8, SY = 16, SZ = 32;
constexpr int kScatterThreads = SY * SZ;
constexpr int kScatterBox = 9728;  // 76 KiB: two workgroups a CU

// Cell and fraction of the warp along one axis; the cell is clamped as in the
// image pass.  (The image pass picks the cell at an exact integer index with
// care, for the one-sided derivative; the weights here do not depend on it.)
template <bool POW2>
__device__ inline void cell(double yhat, double h, double ih, int m, int& i0, float& f) {
    double xi = POW2 ? fma(yhat, ih, -0.5) : yhat / h - 0.5;
    xi = fmin(fmax(xi, 0.0), static_cast<double>(m - 1));
    i0 = min(static_cast<int>(xi), m - 2);
    f = static_cast<float>(xi - static_cast<double>(i0));
}

template <bool POW2>
__global__ __launch_bounds__(kScatterThreads, 4) void k_scatter_T(ImagePassArgs a) {
    __shared__ double box[kScatterBox];
    __shared__ int red[6][kScatterThreads / 64];

    const int t = threadIdx.x;
    const int ntz = (a.mz + SZ - 1) / SZ, nty = (a.my + SY - 1) / SY;
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int z0 = (tile % ntz) * SZ, y0 = ((tile / ntz) % nty) * SY, x0 = tile / (ntz * nty) * SX;
    const int gy = min(y0 + t / SZ, a.my - 1), gz = min(z0 + t % SZ, a.mz - 1);
    const bool in = y0 + t / SZ < a.my && z0 + t % SZ < a.mz;
    const int nx = min(SX, a.mx - x0);

    // the column's cells and fractions
    uint64_t c0[SX];  // packed cell, 21 bits an axis
    float f[SX][3], e[SX];
    int lo[3] = {1 << 30, 1 << 30, 1 << 30}, hi[3] = {0, 0, 0};
    {
        const int64_t plane = static_cast<int64_t>(a.my) * a.mz;
        const float* pe = a.sens + x0 * plane + (static_cast<int64_t>(gy) * a.mz + gz);
#pragma unroll
        for (int k = 0; k < SX; ++k) e[k] = pe[min(k, nx - 1) * plane];
        const int64_t nyz = static_cast<int64_t>(a.ny) * a.nz, Ny = a.nx * nyz;
        const int o = a.j0y[gy] * a.nz + a.j0z[gz];
        const double wy1 = a.w1y[gy], wz1 = a.w1z[gz];
        auto column = [&](int j, double (&u)[3]) {
            const float* p = a.y + min(j, a.nx - 1) * nyz;
            float v[3][4];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                v[c][0] = p[c * Ny + o];
                v[c][1] = p[c * Ny + o + 1];
                v[c][2] = p[c * Ny + o + a.nz];
                v[c][3] = p[c * Ny + o + a.nz + 1];
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const double v0 = v[c][0], v2 = v[c][2];
                const double q0 = fma(wz1, v[c][1] - v0, v0), q1 = fma(wz1, v[c][3] - v2, v2);
                u[c] = fma(wy1, q1 - q0, q0);
            }
        };
        double ulo[3], uhi[3];
        int j = a.j0x[x0];
        column(j, ulo);
        column(j + 1, uhi);
#pragma unroll
        for (int k = 0; k < SX; ++k) {
            const int gx = min(x0 + k, a.mx - 1);
            if (a.j0x[gx] != j) {  // the next node cell (at least two points a cell)
                ++j;
#pragma unroll
                for (int c = 0; c < 3; ++c) ulo[c] = uhi[c];
                column(j + 1, uhi);
            }
            const double wx1 = a.w1x[gx];
            int i[3];
            cell<POW2>(fma(wx1, uhi[0] - ulo[0], ulo[0]), a.hx, a.ihx, a.mx, i[0], f[k][0]);
            cell<POW2>(fma(wx1, uhi[1] - ulo[1], ulo[1]), a.hy, a.ihy, a.my, i[1], f[k][1]);
            cell<POW2>(fma(wx1, uhi[2] - ulo[2], ulo[2]), a.hz, a.ihz, a.mz, i[2], f[k][2]);
            c0[k] = static_cast<uint64_t>(i[0]) << 42 | static_cast<uint64_t>(i[1]) << 21 |
                    static_cast<uint64_t>(i[2]);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                lo[d] = min(lo[d], i[d]);
                hi[d] = max(hi[d], i[d]);
            }
        }
    }
    // the box of cells
#pragma unroll
    for (int d = 0; d < 3; ++d) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            lo[d] = min(lo[d], __shfl_xor(lo[d], o, 64));
            hi[d] = max(hi[d], __shfl_xor(hi[d], o, 64));
        }
        if ((t & 63) == 0) {
            red[d][t >> 6] = lo[d];
            red[3 + d][t >> 6] = hi[d];
        }
    }
    __syncthreads();
    int org[3], ext[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        int l = red[d][0], h = red[3 + d][0];
#pragma unroll
        for (int w = 1; w < kScatterThreads / 64; ++w) {
            l = min(l, red[d][w]);
            h = max(h, red[3 + d][w]);
        }
        org[d] = __builtin_amdgcn_readfirstlane(l);
        ext[d] = __builtin_amdgcn_readfirstlane(h) + 2 - org[d];
    }
    const int64_t vol = static_cast<int64_t>(ext[0]) * ext[1] * ext[2];
    const bool fits = vol <= kScatterBox;
    if (fits) {
        for (int i = t; i < static_cast<int>(vol); i += kScatterThreads) box[i] = 0.0;
        __syncthreads();
    }
    const float gscale = a.gscale != nullptr ? static_cast<float>(*a.gscale) : 1.0f;
    const int row = fits ? ext[2] : a.mz;
    const int64_t slab = fits ? static_cast<int64_t>(ext[1]) * ext[2]
                              : static_cast<int64_t>(a.my) * a.mz;
    auto scatter = [&](auto* G) {
        using V = std::remove_pointer_t<decltype(G)>;
#pragma unroll
        for (int k = 0; k < SX; ++k) {
            if (k >= nx || !in) continue;
            const float es = e[k] * gscale;
            const float fx = f[k][0], fy = f[k][1], fz = f[k][2];
            const float qx = 1.0f - fx, qy = 1.0f - fy, qz = 1.0f - fz;
            const int ix = static_cast<int>(c0[k] >> 42);
            const int iy = static_cast<int>(c0[k] >> 21) & 0x1fffff;
            const int iz = static_cast<int>(c0[k]) & 0x1fffff;
            V* g = fits ? G + ((ix - org[0]) * static_cast<int>(slab) + (iy - org[1]) * row +
                               (iz - org[2]))
                        : G + (ix * slab + static_cast<int64_t>(iy) * row + iz);
            auto put = [&](V* p, float w) {
                atomicAdd(p, static_cast<V>(w * qz));
                atomicAdd(p + 1, static_cast<V>(w * fz));
            };
            put(g, es * qx * qy);
            put(g + row, es * qx * fy);
            put(g + slab, es * fx * qy);
            put(g + slab + row, es * fx * fy);
        }
    };
    if (!fits) {
        scatter(a.gT_atomic);
        return;
    }
    scatter(box);
    __syncthreads();
    // a wave takes rows of the box
    const int rows = ext[0] * ext[1];
    for (int r = __builtin_amdgcn_readfirstlane(t >> 6); r < rows; r += kScatterThreads / 64) {
        const int bx = r / ext[1], by = r - bx * ext[1];
        float* G = a.gT_atomic + (static_cast<int64_t>(org[0] + bx) * a.my + (org[1] + by)) * a.mz +
                   org[2];
        for (int z = t & 63; z < ext[2]; z += 64) {
            const double v = box[r * ext[2] + z];
            if (v != 0.0) atomicAdd(G + z, static_cast<float>(v));
        }
    }
}

}  // namespace

void launch_scatter_T(const ImagePassArgs& a, hipStream_t s) {
    const int64_t nb = int64_t{(a.mx + SX - 1) / SX} * ((a.my + SY - 1) / SY) *
                       ((a.mz + SZ - 1) / SZ);
    const dim3 g(static_cast<unsigned>(nb)), b(kScatterThreads);
    if (a.pow2h)
        hipLaunchKernelGGL(k_scatter_T<true>, g, b, 0, s, a);
    else
        hipLaunchKernelGGL(k_scatter_T<false>, g, b, 0, s, a);
}

}  // namespace ngf
