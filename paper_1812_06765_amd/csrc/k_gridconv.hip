// Standalone grid conversion: y_hat = P y and the three ways of applying P^T
// that Sec. 2.2 ("Grid conversion") compares:
//
// * gather (Eq. 3, the paper's scheme): each deformation node sums
//   omega_x omega_y omega_z z[i] over the index sets of its three axes (the sum
//   along x in registers on the way); every write has one owner;
// * atomic scatter (the earlier GPU scheme): one thread per image point adds
//   its weighted value into the 8 nodes of its cell with atomic additions;
// * red-black slices (the earlier scheme): the image slices of the odd x
//   cells are done in parallel, then those of the even x cells.  A cell's
//   slices reach only the node planes at its two ends, and cells of one
//   parity are two apart, so within a phase no two cells share a node plane;
//   within a cell one thread per (y, z) node sums the slices over its y and
//   z index sets and adds the result to the two node planes (no atomics).
//
// All three compute the same sums (in different orders).  These operators
// are for measurement and testing; the evaluation itself fuses P into the
// warp and P^T into the image and node passes.
#include "ngf_internal.h"

#include <algorithm>

namespace ngf {

namespace {

struct Maps {
    const int32_t* j0[3];
    const float* w0[3];
    const float* w1[3];
    int m[3];
    int n[3];
};

// y_hat = P y (float64 accumulation, float32 result); y, yhat component-major.
// Bound by the 12 bytes a voxel that it writes.  A thread owns one (y, z)
// position of the image plane (taken flat, so any row length fills the waves)
// and walks cx planes along x: y interpolated in its column at the two node
// planes around x stays in registers, a voxel is one interpolation along x,
// and the next node plane is read ahead.  256 x 256 x 192, ratio 2: 39 us, 95
// with a thread a voxel that read its 24 node values; the write alone takes
// 29 us at the rate of a large copy.
__global__ __launch_bounds__(kThreads) void k_apply_P(Maps a, const float* __restrict__ y,
                                                      float* __restrict__ yh, int cx) {
    const int plane = a.m[1] * a.m[2];
    const int64_t N = static_cast<int64_t>(a.m[0]) * plane;
    const int64_t nyz = static_cast<int64_t>(a.n[1]) * a.n[2], Ny = a.n[0] * nyz;
    const int q = blockIdx.x * kThreads + threadIdx.x;
    if (q >= plane) return;
    const int iy = q / a.m[2], iz = q - iy * a.m[2];
    const double wy0 = a.w0[1][iy], wy1 = a.w1[1][iy], wz0 = a.w0[2][iz], wz1 = a.w1[2][iz];
    const double w00 = wy0 * wz0, w01 = wy0 * wz1, w10 = wy1 * wz0, w11 = wy1 * wz1;
    const int o = a.j0[1][iy] * a.n[2] + a.j0[2][iz];
    const int x0 = blockIdx.y * cx, x1 = min(x0 + cx, a.m[0]);
    auto load = [&](int j, float (&v)[3][4]) {
        const float* p = y + min(j, a.n[0] - 1) * nyz;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            v[c][0] = p[c * Ny + o];
            v[c][1] = p[c * Ny + o + 1];
            v[c][2] = p[c * Ny + o + a.n[2]];
            v[c][3] = p[c * Ny + o + a.n[2] + 1];
        }
    };
    auto column = [&](const float (&v)[3][4], double (&u)[3]) {
#pragma unroll
        for (int c = 0; c < 3; ++c)
            u[c] = w00 * v[c][0] + w01 * v[c][1] + w10 * v[c][2] + w11 * v[c][3];
    };
    int j = a.j0[0][x0];
    float v0[3][4], v1[3][4];
    double lo[3], hi[3];
    load(j, v0);
    load(j + 1, v1);
    column(v0, lo);
    column(v1, hi);
    load(j + 2, v0);
    for (int ix = x0; ix < x1; ++ix) {
        if (a.j0[0][ix] != j) {  // the next cell (at least two points a cell)
            ++j;
#pragma unroll
            for (int c = 0; c < 3; ++c) lo[c] = hi[c];
            column(v0, hi);
            load(j + 2, v0);
        }
        const double wx0 = a.w0[0][ix], wx1 = a.w1[0][ix];
        float* out = yh + static_cast<int64_t>(ix) * plane;
#pragma unroll
        for (int c = 0; c < 3; ++c)
            out[c * N + q] = static_cast<float>(wx0 * lo[c] + wx1 * hi[c]);
    }
}

// weight of image index i for node j along one axis (0 outside the index set)
__device__ inline float omega(const Maps& a, int d, int i, int j) {
    const int j0 = a.j0[d][i];
    return j0 == j ? a.w0[d][i] : (j0 + 1 == j ? a.w1[d][i] : 0.0f);
}

// index set of node j along one axis (Eq. 3): the contiguous run of image
// points whose lower node is j - 1 or j, [lo, hi), from the exact integer
// map (no table search)
struct Range {
    int lo, hi;
};
__device__ inline Range omega_range(const Maps& a, int d, int j) {
    return Range{first_at_least(j - 1, a.m[d], a.n[d]), first_at_least(j + 1, a.m[d], a.n[d])};
}

// Gather: a workgroup owns a tile of ny x nz nodes in (y, z) and cx node planes
// and walks the image planes of their index sets.  Bound by the 12 bytes a
// voxel that it reads, so the sum along x is taken first: a thread holds
// kGatherPos positions of the tile's image window (window positions taken
// flat: any width fills the waves), each with the running sums of the two node
// planes around x, and the next plane's values are in flight meanwhile.  Once
// a node plane is complete its sums go to LDS, where a thread per node adds its
// index sets along y and z; the two buffers need one barrier a node plane.
// U: points of an index set along y and z (4 or 8 for ratios 2 and 4, whose
// weights then stay in registers; the cell that an end node does not have reads
// zeros behind the window: one of the set's own values, with weight 0, would make
// an infinity a NaN), 0 where they differ from node to node.
// 256 x 256 x 192: 37 us at ratio 2 and 41 at ratio 4, against 333 and 629 with
// a thread a node that read its whole index set; the read alone takes 29 us.
constexpr int kPBlocks = 2048, kGatherBlocks = 512;
constexpr int kGatherThreads = 512, kGatherPos = 4;
constexpr int kGatherWindow = kGatherThreads * kGatherPos;
struct GatherTile {
    int ny, nz, cx;  // nodes in y and z, node planes a workgroup
    int tz, ty;      // tiles
};

template <int U>
__global__ __launch_bounds__(kGatherThreads) void k_PT_gather(Maps a, GatherTile g,
                                                              const float* __restrict__ z,
                                                              float* __restrict__ out) {
    constexpr int K = kGatherPos;
    __shared__ float win[2][3][kGatherWindow + U / 2];
    const int plane = a.m[1] * a.m[2];
    const int64_t N = static_cast<int64_t>(a.m[0]) * plane;
    const int64_t nyz = static_cast<int64_t>(a.n[1]) * a.n[2], Ny = a.n[0] * nyz;
    const int t = threadIdx.x;
    const int bid = xcd_tile(blockIdx.x, gridDim.x);
    const int bz = bid % g.tz, by = (bid / g.tz) % g.ty, bx = bid / (g.tz * g.ty);
    const int jx0 = bx * g.cx, jx1 = min(jx0 + g.cx, a.n[0]);
    const int jy0 = by * g.ny, jy1 = min(jy0 + g.ny, a.n[1]);
    const int jz0 = bz * g.nz, jz1 = min(jz0 + g.nz, a.n[2]);
    const int iy0 = first_at_least(jy0 - 1, a.m[1], a.n[1]);
    const int iz0 = first_at_least(jz0 - 1, a.m[2], a.n[2]);
    const int wz = first_at_least(jz1, a.m[2], a.n[2]) - iz0;
    const int wy = first_at_least(jy1, a.m[1], a.n[1]) - iy0;
    int off[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int q = min(t + k * kGatherThreads, wy * wz - 1);
        off[k] = (iy0 + q / wz) * a.m[2] + iz0 + q % wz;
    }
    // the thread's node
    const int nzt = jz1 - jz0;
    const int tn = min(t, (jy1 - jy0) * nzt - 1);
    const int jy = jy0 + tn / nzt, jz = jz0 + tn % nzt;
    const bool own = t < (jy1 - jy0) * nzt;
    const Range ry = omega_range(a, 1, jy), rz = omega_range(a, 2, jz);
    float uy[U > 0 ? U : 1], uz[U > 0 ? U : 1];
    if constexpr (U > 0) {
#pragma unroll
        for (int k = 0; k < U; ++k) {
            // beyond the index set (at the grid's ends): weight 0
            uy[k] = ry.lo + k < ry.hi ? omega(a, 1, ry.lo + k, jy) : 0.0f;
            uz[k] = rz.lo + k < rz.hi ? omega(a, 2, rz.lo + k, jz) : 0.0f;
        }
    }
    const int base = (ry.lo - iy0) * wz + (rz.lo - iz0);
    if constexpr (U > 0) {
        constexpr int H = U / 2;
        if (t < 6 * H) win[t / (3 * H)][t / H % 3][kGatherWindow + t % H] = 0.0f;
    }
    int buf = 0;
    float A[3][K] = {}, Bn[3][K] = {}, v[3][K];
    auto load = [&](int ix) {
        const float* p = z + static_cast<int64_t>(ix) * plane;
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int k = 0; k < K; ++k) v[c][k] = p[c * N + off[k]];
    };
    auto emit = [&](int j, const float (&s)[3][K]) {
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int k = 0; k < K; ++k) win[buf][c][t + k * kGatherThreads] = s[c][k];
        __syncthreads();
        if (own) {
            float r[3] = {0.0f, 0.0f, 0.0f};
            if constexpr (U > 0) {
#pragma unroll
                for (int p = 0; p < U; ++p) {
                    // the row's points in the node's first cell and in its second
                    const int first = p < ry.hi - ry.lo ? base + p * wz : kGatherWindow;
                    const int second = p < ry.hi - ry.lo && rz.hi - rz.lo == U ? first + U / 2
                                                                               : kGatherWindow;
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const float *a0 = win[buf][c] + first, *a1 = win[buf][c] + second;
                        float rs = 0.0f;
#pragma unroll
                        for (int q = 0; q < U / 2; ++q) rs = fmaf(uz[q], a0[q], rs);
#pragma unroll
                        for (int q = 0; q < U / 2; ++q) rs = fmaf(uz[U / 2 + q], a1[q], rs);
                        r[c] = fmaf(uy[p], rs, r[c]);
                    }
                }
            } else {
                for (int iy = ry.lo; iy < ry.hi; ++iy) {
                    const float wyi = omega(a, 1, iy, jy);
                    const int row = base + (iy - ry.lo) * wz;
                    float rs[3] = {0.0f, 0.0f, 0.0f};
                    for (int iz = rz.lo; iz < rz.hi; ++iz) {
                        const float wzi = omega(a, 2, iz, jz);
#pragma unroll
                        for (int c = 0; c < 3; ++c)
                            rs[c] = fmaf(wzi, win[buf][c][row + iz - rz.lo], rs[c]);
                    }
#pragma unroll
                    for (int c = 0; c < 3; ++c) r[c] = fmaf(wyi, rs[c], r[c]);
                }
            }
            const int64_t k = j * nyz + static_cast<int64_t>(jy) * a.n[2] + jz;
#pragma unroll
            for (int c = 0; c < 3; ++c) out[c * Ny + k] = r[c];
        }
        buf ^= 1;
    };
    int ix = first_at_least(jx0 - 1, a.m[0], a.n[0]);
    const int last = first_at_least(jx1, a.m[0], a.n[0]) - 1;
    load(ix);
    for (int cell = max(jx0 - 1, 0); cell < min(jx1, a.n[0] - 1); ++cell) {
        const int end = first_at_least(cell + 1, a.m[0], a.n[0]);
        for (; ix < end; ++ix) {
            const float wx0 = a.w0[0][ix], wx1 = a.w1[0][ix];
            float u[3][K];
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int k = 0; k < K; ++k) u[c][k] = v[c][k];
            load(min(ix + 1, last));
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    A[c][k] = fmaf(wx0, u[c][k], A[c][k]);
                    Bn[c][k] = fmaf(wx1, u[c][k], Bn[c][k]);
                }
        }
        if (cell >= jx0) emit(cell, A);
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int k = 0; k < K; ++k) {
                A[c][k] = Bn[c][k];
                Bn[c][k] = 0.0f;
            }
    }
    if (jx1 == a.n[0]) emit(jx1 - 1, A);
}

__global__ __launch_bounds__(kThreads) void k_PT_atomic(Maps a, const float* __restrict__ z,
                                                        float* __restrict__ out) {
    const int64_t N = static_cast<int64_t>(a.m[0]) * a.m[1] * a.m[2];
    const int64_t Ny = static_cast<int64_t>(a.n[0]) * a.n[1] * a.n[2];
    for (int64_t i = blockIdx.x * static_cast<int64_t>(kThreads) + threadIdx.x; i < N;
         i += static_cast<int64_t>(gridDim.x) * kThreads) {
        const int iz = static_cast<int>(i % a.m[2]);
        const int iy = static_cast<int>((i / a.m[2]) % a.m[1]);
        const int ix = static_cast<int>(i / (static_cast<int64_t>(a.m[2]) * a.m[1]));
        const int jx = a.j0[0][ix], jy = a.j0[1][iy], jz = a.j0[2][iz];
        const float wx[2] = {a.w0[0][ix], a.w1[0][ix]};
        const float wy[2] = {a.w0[1][iy], a.w1[1][iy]};
        const float wz[2] = {a.w0[2][iz], a.w1[2][iz]};
        const float v[3] = {z[i], z[N + i], z[2 * N + i]};
        for (int p = 0; p < 2; ++p)
            for (int q = 0; q < 2; ++q)
                for (int r = 0; r < 2; ++r) {
                    const float w = wx[p] * wy[q] * wz[r];
                    const int64_t j =
                        ((jx + p) * static_cast<int64_t>(a.n[1]) + jy + q) * a.n[2] + jz + r;
                    atomicAdd(out + j, w * v[0]);
                    atomicAdd(out + Ny + j, w * v[1]);
                    atomicAdd(out + 2 * Ny + j, w * v[2]);
                }
    }
}

// One phase of the red-black scheme: every x cell gx of parity px, one
// thread per (cell, y node, z node).  The thread sums the cell's slices (the
// image points whose lower x node is gx) over its y and z index sets, each
// slice weighted for node plane gx and for gx + 1, and adds both sums to the
// output; no other thread of the phase touches those nodes.
__global__ __launch_bounds__(kThreads) void k_PT_redblack(Maps a, const float* __restrict__ z,
                                                          float* __restrict__ out, int px) {
    const int64_t N = static_cast<int64_t>(a.m[0]) * a.m[1] * a.m[2];
    const int64_t Ny = static_cast<int64_t>(a.n[0]) * a.n[1] * a.n[2];
    const int cells = (a.n[0] - 1 - px + 1) / 2;  // x cells of this parity
    const int64_t nyz = static_cast<int64_t>(a.n[1]) * a.n[2];
    for (int64_t t = blockIdx.x * static_cast<int64_t>(kThreads) + threadIdx.x;
         t < cells * nyz; t += static_cast<int64_t>(gridDim.x) * kThreads) {
        const int gx = 2 * static_cast<int>(t / nyz) + px;
        const int jy = static_cast<int>((t / a.n[2]) % a.n[1]);
        const int jz = static_cast<int>(t % a.n[2]);
        // the cell's slices: image points with lower x node gx
        const int ilo = first_at_least(gx, a.m[0], a.n[0]);
        const int ihi = first_at_least(gx + 1, a.m[0], a.n[0]);
        const Range ry = omega_range(a, 1, jy), rz = omega_range(a, 2, jz);
        float lo[3] = {0.0f, 0.0f, 0.0f}, hi[3] = {0.0f, 0.0f, 0.0f};
        for (int ix = ilo; ix < ihi; ++ix) {
            const float wx0 = a.w0[0][ix], wx1 = a.w1[0][ix];
            float s[3] = {0.0f, 0.0f, 0.0f};
            for (int iy = ry.lo; iy < ry.hi; ++iy) {
                const float wy = omega(a, 1, iy, jy);
                for (int iz = rz.lo; iz < rz.hi; ++iz) {
                    const float w = wy * omega(a, 2, iz, jz);
                    const int64_t i = (static_cast<int64_t>(ix) * a.m[1] + iy) * a.m[2] + iz;
                    s[0] = fmaf(w, z[i], s[0]);
                    s[1] = fmaf(w, z[N + i], s[1]);
                    s[2] = fmaf(w, z[2 * N + i], s[2]);
                }
            }
            for (int c = 0; c < 3; ++c) {
                lo[c] = fmaf(wx0, s[c], lo[c]);
                hi[c] = fmaf(wx1, s[c], hi[c]);
            }
        }
        const int64_t j = (static_cast<int64_t>(gx) * a.n[1] + jy) * a.n[2] + jz;
        for (int c = 0; c < 3; ++c) {
            out[c * Ny + j] += lo[c];
            out[c * Ny + j + nyz] += hi[c];
        }
    }
}

Maps make_maps(const int32_t* const j0[3], const float* const w0[3], const float* const w1[3],
               const int m[3], const int n[3]) {
    Maps a{};
    for (int d = 0; d < 3; ++d) {
        a.j0[d] = j0[d];
        a.w0[d] = w0[d];
        a.w1[d] = w1[d];
        a.m[d] = m[d];
        a.n[d] = n[d];
    }
    return a;
}

int blocks_for(int64_t n) {
    int64_t b = (n + kThreads - 1) / kThreads;
    return static_cast<int>(b < 1 ? 1 : (b > 65536 ? 65536 : b));
}

// Tile of the gather: as wide as the window's size allows up to 72 image
// points along z (whole lines of 128 bytes and little halo), then as many rows;
// the window holds the at most ceil((nodes + 1) m / (n - 1)) points of its
// nodes' index sets.  Node planes a workgroup for about two workgroups a CU:
// four read more halo planes than they hide (37 -> 44 us at 256 x 256 x 192).
GatherTile gather_tile(const Maps& a) {
    auto points = [&](int d, int nodes) {
        return static_cast<int>((int64_t{nodes + 1} * a.m[d] + a.n[d] - 2) / (a.n[d] - 1));
    };
    auto most = [&](int d, int window) {  // nodes that fit
        int v = 1;
        while (v < a.n[d] && points(d, v + 1) <= window) ++v;
        return v;
    };
    GatherTile g{};
    const int wmax = std::min(72, kGatherWindow / points(1, 1));
    g.tz = (a.n[2] + most(2, wmax) - 1) / most(2, wmax);
    g.nz = (a.n[2] + g.tz - 1) / g.tz;
    const int my = most(1, kGatherWindow / points(2, g.nz));
    g.ty = (a.n[1] + my - 1) / my;
    g.ny = (a.n[1] + g.ty - 1) / g.ty;
    const int64_t tiles = int64_t{g.ty} * g.tz;
    g.cx = static_cast<int>(
        std::max<int64_t>(1, (a.n[0] * tiles + kGatherBlocks - 1) / kGatherBlocks));
    return g;
}

}  // namespace

void launch_apply_P(const int32_t* const j0[3], const float* const w0[3],
                    const float* const w1[3], const int m[3], const int n[3], const float* y,
                    float* yh, hipStream_t s) {
    const Maps a = make_maps(j0, w0, w1, m, n);
    const int64_t cols = (int64_t{m[1]} * m[2] + kThreads - 1) / kThreads;
    // planes a thread: about kPBlocks workgroups (half or twice as many change
    // little), at least 4 planes for the two node planes read first
    const int cx = static_cast<int>(
        std::max<int64_t>(4, std::min<int64_t>(32, m[0] * cols / kPBlocks)));
    hipLaunchKernelGGL(k_apply_P, dim3(static_cast<unsigned>(cols), (m[0] + cx - 1) / cx),
                       dim3(kThreads), 0, s, a, y, yh, cx);
}

// scheme: 0 gather, 1 atomic scatter, 2 red-black.  `out` must be zeroed by
// the caller for schemes 1 and 2.
void launch_apply_PT(const int32_t* const j0[3], const float* const w0[3],
                     const float* const w1[3], const int m[3], const int n[3], const float* z,
                     float* out, int scheme, hipStream_t s) {
    const Maps a = make_maps(j0, w0, w1, m, n);
    const int64_t N = static_cast<int64_t>(m[0]) * m[1] * m[2];
    if (scheme == 0) {
        const GatherTile g = gather_tile(a);
        const int64_t nb = int64_t{g.tz} * g.ty * ((n[0] + g.cx - 1) / g.cx);
        const dim3 gr(static_cast<unsigned>(nb)), b(kGatherThreads);
        auto ratio = [&](int r) {
            return m[1] == r * (n[1] - 1) && m[2] == r * (n[2] - 1);
        };
        if (ratio(2))
            hipLaunchKernelGGL(k_PT_gather<4>, gr, b, 0, s, a, g, z, out);
        else if (ratio(4))
            hipLaunchKernelGGL(k_PT_gather<8>, gr, b, 0, s, a, g, z, out);
        else
            hipLaunchKernelGGL(k_PT_gather<0>, gr, b, 0, s, a, g, z, out);
    } else if (scheme == 1) {
        hipLaunchKernelGGL(k_PT_atomic, dim3(blocks_for(N)), dim3(kThreads), 0, s, a, z, out);
    } else {
        // odd x cells, then even ones (the second phase starts after the
        // first on the stream: they share node planes)
        const int64_t nyz = static_cast<int64_t>(n[1]) * n[2];
        for (int px = 1; px >= 0; --px) {
            const int64_t cells = (n[0] - 1 - px + 1) / 2;
            hipLaunchKernelGGL(k_PT_redblack, dim3(blocks_for(cells * nyz)), dim3(kThreads), 0, s,
                               a, z, out, px);
        }
    }
}

}  // namespace ngf
