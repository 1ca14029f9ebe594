// Float64 evaluation of J and grad J (Eq. 1-3), for the precision study.
//
// The production evaluation keeps the bulk arithmetic in float32 (Sec. 2.2
// computes in single precision) and fuses every image-grid step into one
// pass.  This file computes the same objective with every value in float64,
// over the image and node grids, so that the effect of float32 can be measured
// on the device against a float64 run of the same method:
//
//   k64_warp     P y (trilinear, exact rational weights), the warp T(P y) and
//                its derivative with respect to y_hat           per voxel
//                and, in blocks of their own, A u for u = y - X (seven-point,
//                replicated ghost nodes), partial sums of (A u)^2 per node
//   k64_ngf      central differences of T_y and R, the NGF terms (Eq. 2),
//                v = dD/d(grad T_y), partial sums of 1 - r^2     per voxel
//   k64_gather   e = sum_d G_d^T v_d and z = e dT_y/dy_hat per voxel, P^T z
//                (Eq. 3, gather over the index sets) plus alpha hbar^y A (A u)
//                per node
//   k64_reduce   D, S and J from the partial sums in a fixed order
//
// Intermediates live in one float64 scratch buffer of the context:
// T_y (N), dT_y/dy_hat (3N), v (3N), A u (3 N^y) and the partial sums.  Every
// reduction has a fixed order, so equal inputs give equal outputs.
//
// The voxel kernels walk along x: a thread owns one (y, z) position of the image
// plane (taken flat), whose index maps it looks up once, and cx planes.  The
// grid has a wave for every few planes, since each is a chain of dependent
// loads.  128 x 112 x 96: k64_warp 22 us, k64_ngf 16 and k64_gather 34, against 37
// + 9, 19 and 79 as kernels with a thread a voxel or node that looked its place
// and every weight up by 64-bit divisions.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>

#include "../../include/ngfreg.h"
#include "ngf_ctx.h"
#include "ngf_internal.h"

namespace {

using namespace ngf;

constexpr int kT = 256;       // threads per workgroup
constexpr int kChunk = 32;    // image planes a workgroup walks, at most
constexpr int kSlots64 = 1024;  // workgroups the voxel kernels aim at

struct Grid64 {
    int m[3], my[3];
    double h[3], hy[3];
    double ih[3];    // 1 / h
    double h2[3], i2h[3];     // 2 h and its reciprocal
    double hy2[3], ihy2[3];  // hy^2 and its reciprocal
    int64_t n, ny;
    int pow2h;       // every 1 / h is exact
    int cx;          // image planes a workgroup
    int cols;        // workgroups across the image plane
};

// Sum over the workgroup in a fixed order; the result in thread 0.
template <int NT>
__device__ inline double block_sum(double v, double* s) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = v;
    __syncthreads();
    double r = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < NT / 64; ++w) r += s[w];
    return r;
}

// Index map of one axis (Sec. 2.2, "Grid conversion"): image point i lies at
// node coordinate num/den, num = (2i+1)(m^y-1), den = 2m; node j0 = num div
// den takes weight (den - r)/den and node j0+1 weight r/den, r = num mod den.
// (32-bit for m <= 32768, which the pyramid's limits ensure.)
__device__ inline void index_map(int i, int m, int my, int& j0, double& w0, double& w1) {
    const int num = (2 * i + 1) * (my - 1);
    const int den = 2 * m;
    const int r = num % den;
    j0 = num / den;
    w1 = static_cast<double>(r) / static_cast<double>(den);
    w0 = static_cast<double>(den - r) / static_cast<double>(den);
}

// Quotient by 2 h along an axis.
__device__ inline double over_2h(const Grid64& g, double v, int d) {
    return quotient(v, g.h2[d], g.i2h[d]);
}

// Displacement u = y - X at node (j) of component c, X_d = j_d h^y_d.
__device__ inline double disp(const double* yc, const Grid64& g, const int j[3], int c) {
    const int64_t k = (static_cast<int64_t>(j[0]) * g.my[1] + j[1]) * g.my[2] + j[2];
    return yc[k] - j[c] * g.hy[c];
}

// Seven-point Laplacian with replicated ghost nodes of a node field given by
// a functor value(j).
template <class F>
__device__ inline double laplacian(const Grid64& g, const int j[3], F value) {
    const double u0 = value(j);
    double out = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        int jp[3] = {j[0], j[1], j[2]}, jm[3] = {j[0], j[1], j[2]};
        jp[d] = min(j[d] + 1, g.my[d] - 1);
        jm[d] = max(j[d] - 1, 0);
        out += quotient_with_infinities(value(jp) - 2.0 * u0 + value(jm), g.hy2[d], g.ihy2[d]);
    }
    return out;
}

// A u for u = y - X, every component, at the nodes of one workgroup; its
// partial sum of (A u)^2.
__device__ inline void lap_block(const Grid64& g, const double* __restrict__ y,
                                 double* __restrict__ Au, double* __restrict__ spart, int block,
                                 double* red) {
    const uint32_t n = static_cast<uint32_t>(block) * kT + threadIdx.x;
    double acc = 0.0;
    if (n < g.ny) {
        const uint32_t nz = g.my[2], ny = g.my[1], t = n / nz;
        const int j[3] = {static_cast<int>(t / ny), static_cast<int>(t % ny),
                          static_cast<int>(n - t * nz)};
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double* yc = y + c * g.ny;
            const double a = laplacian(g, j, [&](const int* q) { return disp(yc, g, q, c); });
            Au[c * g.ny + n] = a;
            acc += a * a;
        }
    }
    const double s = block_sum<kT>(acc, red);
    if (threadIdx.x == 0) spart[block] = s;
}

// y_hat = P y at one voxel, then the clamped trilinear warp of T there and
// its derivative with respect to y_hat (slope 0 where a coordinate left the
// domain; the cell is clamped to [0, m-2] so the top edge is left-sided).
// The node values of the column stay in registers while x is in one node cell.
// Blocks from `first` on: see lap_block.
template <bool GRAD>
__global__ __launch_bounds__(kT) void k64_warp(Grid64 g, const double* __restrict__ y,
                                               const float* __restrict__ T,
                                               double* __restrict__ Ty, double* __restrict__ dT,
                                               double* __restrict__ Au,
                                               double* __restrict__ spart, int first) {
    __shared__ double red[kT / 64];
    __shared__ double sx[kChunk][2];
    __shared__ int sj[kChunk];
    if (static_cast<int>(blockIdx.x) >= first) {
        lap_block(g, y, Au, spart, blockIdx.x - first, red);
        return;
    }
    const int plane = g.m[1] * g.m[2];
    const int q = (blockIdx.x % g.cols) * kT + threadIdx.x;
    const int x0 = (blockIdx.x / g.cols) * g.cx, x1 = min(x0 + g.cx, g.m[0]);
    if (static_cast<int>(threadIdx.x) < x1 - x0)
        index_map(x0 + threadIdx.x, g.m[0], g.my[0], sj[threadIdx.x], sx[threadIdx.x][0],
                  sx[threadIdx.x][1]);
    __syncthreads();
    if (q >= plane) return;
    int jy, jz;
    double wy[2], wz[2];
    index_map(q / g.m[2], g.m[1], g.my[1], jy, wy[0], wy[1]);
    index_map(q % g.m[2], g.m[2], g.my[2], jz, wz[0], wz[1]);
    const double* col = y + (static_cast<int64_t>(jy) * g.my[2] + jz);
    const int64_t nyz = static_cast<int64_t>(g.my[1]) * g.my[2];
    double v[3][2][4];
    auto load = [&](int j, int a) {
        const double* p = col + j * nyz;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            v[c][a][0] = p[c * g.ny];
            v[c][a][1] = p[c * g.ny + 1];
            v[c][a][2] = p[c * g.ny + g.my[2]];
            v[c][a][3] = p[c * g.ny + g.my[2] + 1];
        }
    };
    int jx = sj[0];
    load(jx, 0);
    load(jx + 1, 1);
    for (int x = x0; x < x1; ++x) {
        const int j = __builtin_amdgcn_readfirstlane(sj[x - x0]);
        if (j != jx) {  // the next node cell (at least two points a cell)
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int k = 0; k < 4; ++k) v[c][0][k] = v[c][1][k];
            jx = j;
            load(jx + 1, 1);
        }
        double w[2][4];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int k = 0; k < 4; ++k) w[a][k] = (sx[x - x0][a] * wy[k >> 1]) * wz[k & 1];
        int i0[3];
        double f[3], s[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            double yh = 0.0;
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int k = 0; k < 4; ++k) yh += w[a][k] * v[d][a][k];
            // with a power-of-two spacing the product rounds like the quotient
            double xi = (g.pow2h ? yh * g.ih[d] : yh / g.h[d]) - 0.5;
            const double top = static_cast<double>(g.m[d] - 1);
            s[d] = (xi >= 0.0 && xi <= top) ? g.ih[d] : 0.0;
            xi = fmin(fmax(xi, 0.0), top);
            i0[d] = min(static_cast<int>(floor(xi)), g.m[d] - 2);
            f[d] = xi - i0[d];
        }
        const float* Tb = T + (static_cast<int64_t>(i0[0]) * plane + i0[1] * g.m[2] + i0[2]);
        const float t8[8] = {Tb[0],     Tb[1],         Tb[g.m[2]],         Tb[g.m[2] + 1],
                             Tb[plane], Tb[plane + 1], Tb[plane + g.m[2]], Tb[plane + g.m[2] + 1]};
        double ty = 0.0, dt[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            const double wa = a ? f[0] : 1.0 - f[0], da = a ? 1.0 : -1.0;
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const double wb = b ? f[1] : 1.0 - f[1], db = b ? 1.0 : -1.0;
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const double wc = e ? f[2] : 1.0 - f[2], dc = e ? 1.0 : -1.0;
                    const double val = static_cast<double>(t8[4 * a + 2 * b + e]);
                    ty += wa * wb * wc * val;
                    dt[0] += da * wb * wc * val;
                    dt[1] += wa * db * wc * val;
                    dt[2] += wa * wb * dc * val;
                }
            }
        }
        const int64_t n = static_cast<int64_t>(x) * plane + q;
        Ty[n] = ty;
        if (GRAD) {
#pragma unroll
            for (int d = 0; d < 3; ++d) dT[d * g.n + n] = dt[d] * s[d];
        }
    }
}

// NGF terms of Eq. 2 at every voxel; v = dD/d(grad T_y) and per-workgroup
// partial sums of 1 - r^2.  Central differences with replicated ghost cells;
// those along x are between the planes in the thread's registers.
template <bool GRAD>
__global__ __launch_bounds__(kT) void k64_ngf(Grid64 g, const double* __restrict__ Ty,
                                              const float* __restrict__ R, double tau,
                                              double rho, double hbar, double* __restrict__ v,
                                              double* __restrict__ dpart) {
    __shared__ double red[kT / 64];
    const int plane = g.m[1] * g.m[2];
    const int qt = (blockIdx.x % g.cols) * kT + threadIdx.x;
    const int x0 = (blockIdx.x / g.cols) * g.cx, x1 = min(x0 + g.cx, g.m[0]);
    const int q = min(qt, plane - 1);
    const int iy = q / g.m[2], iz = q - iy * g.m[2];
    const int yp = iy < g.m[1] - 1 ? g.m[2] : 0, ym = iy > 0 ? -g.m[2] : 0;
    const int zp = iz < g.m[2] - 1 ? 1 : 0, zm = iz > 0 ? -1 : 0;
    auto at = [&](int x) {
        return static_cast<int64_t>(min(max(x, 0), g.m[0] - 1)) * plane + q;
    };
    int64_t n = at(x0);
    double T0 = Ty[at(x0 - 1)], T1 = Ty[n];
    float R0 = R[at(x0 - 1)], R1 = R[n];
    double acc = 0.0;
    for (int x = x0; x < x1; ++x) {
        const int64_t np = at(x + 1);
        const double T2 = Ty[np];
        const float R2 = R[np];
        const double gT[3] = {over_2h(g, T2 - T0, 0), over_2h(g, Ty[n + yp] - Ty[n + ym], 1),
                              over_2h(g, Ty[n + zp] - Ty[n + zm], 2)};
        auto dR = [](float p, float m) { return static_cast<double>(p) - static_cast<double>(m); };
        const double gR[3] = {over_2h(g, dR(R2, R0), 0), over_2h(g, dR(R[n + yp], R[n + ym]), 1),
                              over_2h(g, dR(R[n + zp], R[n + zm]), 2)};
        const double nT = sqrt(gT[0] * gT[0] + gT[1] * gT[1] + gT[2] * gT[2] + tau * tau);
        const double nR = sqrt(gR[0] * gR[0] + gR[1] * gR[1] + gR[2] * gR[2] + rho * rho);
        const double c = gT[0] * gR[0] + gT[1] * gR[1] + gT[2] * gR[2] + tau * rho;
        const double r = c / (nT * nR);
        if (qt < plane) {
            acc += 1.0 - r * r;
            if (GRAD) {
                const double k = -hbar * r / (nT * nR);
                const double p = c / (nT * nT);
#pragma unroll
                for (int d = 0; d < 3; ++d) v[d * g.n + n] = k * (gR[d] - p * gT[d]);
            }
        }
        T0 = T1;
        T1 = T2;
        R0 = R1;
        R1 = R2;
        n = np;
    }
    const double s = block_sum<kT>(acc, red);
    if (threadIdx.x == 0) dpart[blockIdx.x] = s;
}

// grad J: e = sum_d G_d^T v_d (the adjoint of the clamped central difference:
// (w[i-1] - w[i+1])/(2h), with a mirrored ghost -w at the domain's ends) and
// z = e dT_y/dy_hat at the voxels, and at every node P^T z (Eq. 3: the image
// points of the index sets Omega_x x Omega_y x Omega_z, each weighted by the
// product of its per-axis weights toward this node) plus alpha hbar^y A (A u).
// The form of the float32 gather (see GatherTile): a workgroup owns a tile of
// nodes in (y, z) and g.cx node planes and walks the image planes of their
// index sets, the sum along x first, in registers; a completed node plane goes
// to LDS and is summed along y and z there.  One position a thread: with two,
// fewer waves hide the loads (760 -> 844 us for the evaluation of 256^3).
// kGSlots: workgroups aimed at; 256 take 15 % longer at 128 x 112 x 96 (chains of
// more planes), 768 at 256^3 (more halo planes).
constexpr int kGSlots = 512;
constexpr int kGThreads = 1024, kGWindow = kGThreads, kGAxis = 256;
struct Tile64 {
    int ny, nz, cx, ty, tz;  // nodes in y and z, node planes, tiles
};

__global__ __launch_bounds__(kGThreads, 4) void k64_gather(
    Grid64 g, Tile64 tl, const double* __restrict__ v, const double* __restrict__ dT,
    const double* __restrict__ Au, double ahbary, double* __restrict__ grad) {
    __shared__ double win[2][3][kGWindow];
    __shared__ double sw[2][kGAxis][2];  // weights of the window's rows and columns
    __shared__ double sx[kGAxis][2];     // and of the image planes walked
    __shared__ int sj[2][kGAxis];
    __shared__ int sr[2][kGAxis];  // index set of a node: first point, points << 16
    const int plane = g.m[1] * g.m[2];
    const int64_t nyz = static_cast<int64_t>(g.my[1]) * g.my[2];
    const int t = threadIdx.x;
    const int bid = xcd_tile(blockIdx.x, gridDim.x);
    const int bz = bid % tl.tz, by = (bid / tl.tz) % tl.ty, bx = bid / (tl.tz * tl.ty);
    const int jx0 = bx * tl.cx, jx1 = min(jx0 + tl.cx, g.my[0]);
    const int jy0 = by * tl.ny, jy1 = min(jy0 + tl.ny, g.my[1]);
    const int jz0 = bz * tl.nz, jz1 = min(jz0 + tl.nz, g.my[2]);
    const int iy0 = first_at_least(jy0 - 1, g.m[1], g.my[1]);
    const int iz0 = first_at_least(jz0 - 1, g.m[2], g.my[2]);
    const int wy = first_at_least(jy1, g.m[1], g.my[1]) - iy0;
    const int wz = first_at_least(jz1, g.m[2], g.my[2]) - iz0;
    if (t < wy) index_map(iy0 + t, g.m[1], g.my[1], sj[0][t], sw[0][t][0], sw[0][t][1]);
    if (t < wz) index_map(iz0 + t, g.m[2], g.my[2], sj[1][t], sw[1][t][0], sw[1][t][1]);
    int ix = first_at_least(jx0 - 1, g.m[0], g.my[0]);
    const int ix0 = ix, nix = first_at_least(jx1, g.m[0], g.my[0]) - ix0;
    if (t < nix) {
        int jx;
        index_map(ix0 + t, g.m[0], g.my[0], jx, sx[t][0], sx[t][1]);
    }
    auto range = [&](int j, int d, int i0) {
        const int lo = first_at_least(j - 1, g.m[d], g.my[d]);
        return (lo - i0) | (first_at_least(j + 1, g.m[d], g.my[d]) - lo) << 16;
    };
    if (t < jy1 - jy0) sr[0][t] = range(jy0 + t, 1, iy0);
    if (t < jz1 - jz0) sr[1][t] = range(jz0 + t, 2, iz0);
    // the thread's position, its neighbours in the plane, and which of those are
    // mirrored at the domain's ends
    const int wq = min(t, wy * wz - 1);
    const int iy = iy0 + wq / wz, iz = iz0 + wq % wz;
    const int off = iy * g.m[2] + iz;
    const bool ylo = iy == 0, yup = iy == g.m[1] - 1, zlo = iz == 0, zup = iz == g.m[2] - 1;
    const int oym = ylo ? off : off - g.m[2], oyp = yup ? off : off + g.m[2];
    const int ozm = zlo ? off : off - 1, ozp = zup ? off : off + 1;
    const int nzt = jz1 - jz0, nn = (jy1 - jy0) * nzt;
    int buf = 0;
    double A[3] = {}, Bn[3] = {};
    auto emit = [&](int jx, const double (&sum)[3]) {
#pragma unroll
        for (int c = 0; c < 3; ++c) win[buf][c][t] = sum[c];
        __syncthreads();
        for (int i = t; i < 3 * nn; i += kGThreads) {
            const int c = i / nn, r = i - c * nn;
            const int ry = r / nzt, rz = r - ry * nzt;
            const int j[3] = {jx, jy0 + ry, jz0 + rz};
            const int ylo = sr[0][ry] & 0xffff, yhi = ylo + (sr[0][ry] >> 16);
            const int zlo = sr[1][rz] & 0xffff, zhi = zlo + (sr[1][rz] >> 16);
            double gd = 0.0;
            for (int y = ylo; y < yhi; ++y) {
                double rs = 0.0;
                for (int z = zlo; z < zhi; ++z)
                    rs += sw[1][z][sj[1][z] == j[2] ? 0 : 1] * win[buf][c][y * wz + z];
                gd += sw[0][y][sj[0][y] == j[1] ? 0 : 1] * rs;
            }
            const double* ac = Au + c * g.ny;
            const double gs = laplacian(g, j, [&](const int* q) {
                return ac[(static_cast<int64_t>(q[0]) * g.my[1] + q[1]) * g.my[2] + q[2]];
            });
            grad[c * g.ny + jx * nyz + static_cast<int64_t>(j[1]) * g.my[2] + j[2]] =
                gd + ahbary * gs;
        }
        buf ^= 1;
    };
    double w[8];  // of plane ix: v_x a plane on, v_y and v_z beside, dT
    auto load = [&](int x) {
        const double* p = v + static_cast<int64_t>(x) * plane;
        const double* d = dT + static_cast<int64_t>(x) * plane;
        w[0] = p[off + (x == g.m[0] - 1 ? 0 : plane)];
        w[1] = p[g.n + oym];
        w[2] = p[g.n + oyp];
        w[3] = p[2 * g.n + ozm];
        w[4] = p[2 * g.n + ozp];
#pragma unroll
        for (int c = 0; c < 3; ++c) w[5 + c] = d[c * g.n + off];
    };
    double vx1 = v[static_cast<int64_t>(ix) * plane + off];
    double vx0 = ix > 0 ? v[static_cast<int64_t>(ix - 1) * plane + off] : -vx1;
    load(ix);
    __syncthreads();
    for (int cell = max(jx0 - 1, 0); cell < min(jx1, g.my[0] - 1); ++cell) {
        const int end = first_at_least(cell + 1, g.m[0], g.my[0]);
        for (; ix < end; ++ix) {
            const double wx0 = sx[ix - ix0][0], wx1 = sx[ix - ix0][1];
            const double ey = (ylo ? -w[1] : w[1]) - (yup ? -w[2] : w[2]);
            const double ez = (zlo ? -w[3] : w[3]) - (zup ? -w[4] : w[4]);
            const double vx2 = ix == g.m[0] - 1 ? -w[0] : w[0];
            const double e = over_2h(g, vx0 - vx2, 0) + over_2h(g, ey, 1) + over_2h(g, ez, 2);
            vx0 = vx1;
            vx1 = w[0];
            double z[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) z[c] = e * w[5 + c];
            load(min(ix + 1, ix0 + nix - 1));
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                A[c] += wx0 * z[c];
                Bn[c] += wx1 * z[c];
            }
        }
        if (cell >= jx0) emit(cell, A);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            A[c] = Bn[c];
            Bn[c] = 0.0;
        }
    }
    if (jx1 == g.my[0]) emit(jx1 - 1, A);
}

Tile64 gather_tile(const Grid64& g) {
    auto points = [&](int d, int nodes) {  // image points of the nodes' index sets, at most
        return static_cast<int>((int64_t{nodes + 1} * g.m[d] + g.my[d] - 2) / (g.my[d] - 1));
    };
    auto most = [&](int d, int window) {
        int n = 1;
        while (n < g.my[d] && points(d, n + 1) <= window) ++n;
        return n;
    };
    Tile64 t{};
    const int nz = most(2, std::min(40, kGWindow / points(1, 1)));
    t.tz = (g.my[2] + nz - 1) / nz;
    t.nz = (g.my[2] + t.tz - 1) / t.tz;
    const int ny = most(1, std::min(kGAxis, kGWindow / points(2, t.nz)));
    t.ty = (g.my[1] + ny - 1) / ny;
    t.ny = (g.my[1] + t.ty - 1) / t.ty;
    // kGSlots workgroups, the planes walked within the table of their weights
    t.cx = static_cast<int>(std::min<int64_t>(
        most(0, kGAxis), (int64_t{g.my[0]} * t.ty * t.tz + kGSlots - 1) / kGSlots));
    return t;
}

// D = (hbar/2) sum(1 - r^2), S = (hbar^y/2) sum (A u)^2, J = D + alpha S, from
// the partial sums of each, in a fixed order.  out = {J, D, S}.
__global__ __launch_bounds__(kT) void k64_reduce(const double* __restrict__ dpart, int nd,
                                                 const double* __restrict__ spart, int ns,
                                                 double half_hbar, double half_hbary,
                                                 double alpha, double* __restrict__ out,
                                                 double* __restrict__ host) {
    __shared__ double red[2][kT / 64];
    double a = 0.0, b = 0.0;
#pragma unroll 4
    for (int k = threadIdx.x; k < nd; k += kT) a += dpart[k];
#pragma unroll 4
    for (int k = threadIdx.x; k < ns; k += kT) b += spart[k];
    const double sd = block_sum<kT>(a, red[0]), ss = block_sum<kT>(b, red[1]);
    if (threadIdx.x == 0) {
        const double D = half_hbar * sd, S = half_hbary * ss;
        out[0] = D + alpha * S;
        out[1] = D;
        out[2] = S;
        if (host) {  // pinned: no copy kernel behind this one
            host[0] = out[0];
            host[1] = D;
            host[2] = S;
        }
    }
}

}  // namespace

using namespace ngf_host;

#define F64CHK(ctx, expr)                                                              \
    do {                                                                               \
        hipError_t e_ = (expr);                                                        \
        if (e_ != hipSuccess)                                                          \
            return fail(ctx, NGF_E_HIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

extern "C" ngf_status ngf_eval_J_grad_f64(ngf_ctx* c, int32_t level, const double* y, double* J,
                                          double* grad, double* DS) {
    if (!c) return NGF_E_ARG;
    if (c->lv.empty()) return fail(c, NGF_E_STATE, "no pyramid");
    if (level < 0 || level >= static_cast<int>(c->lv.size()))
        return fail(c, NGF_E_LEVEL, "bad level");
    if (!y) return fail(c, NGF_E_ARG, "null y");
    const Level& L = c->lv[level];
    Grid64 g{};
    for (int d = 0; d < 3; ++d) {
        g.m[d] = L.m[d];
        g.my[d] = L.my[d];
        g.h[d] = L.h[d];
        g.hy[d] = L.hy[d];
        g.ih[d] = 1.0 / L.h[d];
        g.h2[d] = 2.0 * L.h[d];
        g.i2h[d] = 1.0 / g.h2[d];
        g.hy2[d] = L.hy[d] * L.hy[d];
        g.ihy2[d] = 1.0 / g.hy2[d];
    }
    g.n = L.N();
    g.ny = L.Ny();
    g.pow2h = pow2(L.h[0]) && pow2(L.h[1]) && pow2(L.h[2]);
    g.cols = static_cast<int>((int64_t{g.m[1]} * g.m[2] + kT - 1) / kT);
    g.cx = static_cast<int>(std::max<int64_t>(
        4, std::min<int64_t>(kChunk, int64_t{g.m[0]} * g.cols / kSlots64)));
    const int64_t nvox = int64_t{g.cols} * ((g.m[0] + g.cx - 1) / g.cx);
    const int64_t nlap = (g.ny + kT - 1) / kT;
    // scratch: T_y, dT, v, A u, two sets of partial sums, {J, D, S}
    const size_t need = static_cast<size_t>(7 * g.n + 3 * g.ny + nvox + nlap + 3);
    if (need > c->f64_cap) {
        F64CHK(c, hipStreamSynchronize(c->stream));  // queued work may use the old buffer
        if (c->f64) (void)hipFree(c->f64);
        c->f64 = nullptr;
        c->f64_cap = 0;
        if ((c->faults & NGF_FAULT_ALLOC) ||
            hipMalloc(reinterpret_cast<void**>(&c->f64), need * sizeof(double)) != hipSuccess) {
            (void)hipGetLastError();
            c->f64 = nullptr;
            return fail(c, NGF_E_OOM, "hipMalloc of the float64 scratch failed");
        }
        c->f64_cap = need;
    }
    double* Ty = c->f64;
    double* dT = Ty + g.n;
    double* v = dT + 3 * g.n;
    double* Au = v + 3 * g.n;
    double* dpart = Au + 3 * g.ny;
    double* spart = dpart + nvox;
    double* out = spart + nlap;
    const double hbar = L.h[0] * L.h[1] * L.h[2];
    const double hbary = L.hy[0] * L.hy[1] * L.hy[2];
    hipStream_t s = c->stream;
    const int nv = static_cast<int>(nvox), nl = static_cast<int>(nlap);
    if (grad) {
        const Tile64 tl = gather_tile(g);
        const int nb = tl.ty * tl.tz * ((g.my[0] + tl.cx - 1) / tl.cx);
        k64_warp<true><<<nv + nl, kT, 0, s>>>(g, y, L.T, Ty, dT, Au, spart, nv);
        k64_ngf<true><<<nv, kT, 0, s>>>(g, Ty, L.R, c->p.tau, c->p.rho, hbar, v, dpart);
        k64_gather<<<nb, kGThreads, 0, s>>>(g, tl, v, dT, Au, c->p.alpha * hbary, grad);
    } else {
        k64_warp<false><<<nv + nl, kT, 0, s>>>(g, y, L.T, Ty, dT, Au, spart, nv);
        k64_ngf<false><<<nv, kT, 0, s>>>(g, Ty, L.R, c->p.tau, c->p.rho, hbar, v, dpart);
    }
    k64_reduce<<<1, kT, 0, s>>>(dpart, nv, spart, nl, 0.5 * hbar, 0.5 * hbary, c->p.alpha, out,
                               J || DS ? c->host_jds : nullptr);
    F64CHK(c, hipGetLastError());
    if (J || DS) {
        const double* h3 = c->host_jds;
        F64CHK(c, hipStreamSynchronize(s));
        if (J) *J = h3[0];
        if (DS) {
            DS[0] = h3[1];
            DS[1] = h3[2];
        }
        if (!std::isfinite(h3[0])) return fail(c, NGF_E_NONFINITE, "J is not finite");
    }
    return NGF_OK;
}
