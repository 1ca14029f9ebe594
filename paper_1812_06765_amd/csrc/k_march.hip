// Image-grid pass, marching form.  Same arithmetic as k_image_pass (P and the
// warp with float64 coordinates, NGF term of Eq. 2, its adjoint stencil, the
// tile-local part of the P^T gather of Eq. 3), organised for fewer redundant
// voxels: a workgroup owns a (y, z) tile of TY x TZ voxels and a chunk of CX
// planes along x (the slowest axis) and walks the planes in order, keeping
// rolling planes in LDS.  Halos then exist only inside a plane (two voxels
// for the warped template, one for v) plus four planes per chunk, instead of
// in all three directions.
//
// Per step (plane p_w enters), everything read from LDS was written in an
// earlier step, so one barrier a step suffices:
//   W  P and the warp of plane p_w on the tile, and on the in-plane halo where
//      a later stage reads it; R of the plane beside it
//   V  NGF on plane p_v = p_w - 1: D term, v.  Differences along x, and along
//      y within a thread's pair of rows, are between its own registers
//   E  adjoint on plane p_e = p_w - 2: e = G^T v, dD/dy_hat = e dT, and P^T
//      along y (the pair) and x (two node planes' accumulators) in registers
//   a completed node plane: P^T along z over neighbouring lanes, into LDS; a
//      step later its nodes are summed and stored
// Ghost planes of the x adjoint stencil (x = -1, x = m_x) are not computed:
// E substitutes v_x(-1) = -v_x(0) and v_x(m_x) = -v_x(m_x - 1) directly.
//
// The P^T partial sums are written in the tile layout the node pass reads:
// tile (chunk, ty, tz) owns node block [x0/R, x0/R + CX/R] x [...] x [...].
//
// What bounds it: vector instruction issue.  At 256^3 a voxel takes 228 vector
// instructions, one of which issues in 60 % of the quad-cycles, and the float64 P
// and template index, their largest part, take more than one each.  Two rows of
// one node cell a thread share the z interpolations of P (21 float64
// instructions a pair instead of 36), half the y neighbours and the y part of
// P^T; the halo's positions and offsets stay packed in registers; values are
// settled where they are formed, so that 128 registers suffice (four waves per
// SIMD): 127 and no spill at ratio 2, one spilled register in the 32 x 32 tile's
// gradient forms at ratio 4 and in one of 16 x 64.  256^3, ratio 2, per launch
// at a smooth deformation: 161 us, against 232 and 317 instructions for the
// five-stage form with one voxel's halves in different barriers that this
// replaced (ratio 4: 220 -> 140 us; spacing 0.9: 253 -> 168 us).
#include "ngf_internal.h"

#include <math.h>

#include <atomic>
#include <type_traits>

namespace ngf {

namespace {

__device__ inline int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// Raw buffer access to R, T and y: byte offsets in 32 bits (the host keeps
// the images below 2^30 voxels), the uniform part of an offset in a scalar
// register, no 64-bit address arithmetic per load.  A load past the buffer
// size returns 0 instead of faulting.
__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const float* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, bytes, 0x00020000);
}
__device__ inline float bload(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
__device__ inline void bstore(__amdgpu_buffer_rsrc_t r, float v, uint32_t voff, uint32_t soff) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(v), r, voff, soff, 0);
}
__device__ inline float2 bload2(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
    return make_float2(__uint_as_float(v[0]), __uint_as_float(v[1]));
}

__device__ inline double wave_sum(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    return v;
}

// TY x TZ: the (y, z) tile of a workgroup.  Thread t owns the two voxels
// (2 (t / TZ), t % TZ) and (2 (t / TZ) + 1, t % TZ) of every plane: a pair of
// rows lies in one node cell along y, so the pair shares its interpolation
// along z, its neighbour along y is in the thread's own registers, and the y
// part of P^T is a sum of two registers.
template <int TY, int TZ, int R>
struct March {
    static constexpr int NT = TY * TZ / 2;
    static constexpr int H2Y = TY + 4, H2Z = TZ + 4, NH2 = H2Y * H2Z;
    static constexpr int NFACE = 2 * (TY + TZ);  // faces of the one-voxel halo
    static constexpr int NRING = 2 * NFACE + 4;  // every halo position a stencil reads
    static constexpr int BY = TY / R, BZ = TZ / R, PY = BY + 1, PZ = BZ + 1;
    static constexpr int NQY = TY / R + 3, NQZ = TZ / R + 3, NQ = NQY * NQZ;
    static constexpr int KQ = (3 * NQ + NT - 1) / NT;
    static constexpr int VYS = (TY + 2) * TZ, VZS = TY * (TZ + 2);
    // LDS layout (floats); the node planes hold doubles and come first
    static constexpr int OFF_TY = 12 * NQ;          // after 2 x 3 NQ doubles: 2 x NH2
    static constexpr int OFF_R = OFF_TY + 2 * NH2;  // 2 x NH2
    static constexpr int OFF_VY = OFF_R + 2 * NH2;  // 2 x VYS (gradient form only from here)
    static constexpr int OFF_VZ = OFF_VY + 2 * VYS; // 2 x VZS
    static constexpr int OFF_G = OFF_VZ + 2 * VZS;  // 6 x NT
    static constexpr int LDS_VALUE = OFF_VY, LDS_GRAD = OFF_G + 6 * NT;
    static_assert(TY % 4 == 0 && TZ % 4 == 0 && NT % 64 == 0, "pairs of rows, quads of columns");
    static_assert(TY % R == 0 && TZ % R == 0 && (R == 2 || R == 4), "ratio-aligned tile");
    static_assert(NRING <= NT && PY * PZ <= NT, "one halo position, one node a thread");
    static_assert((LDS_GRAD * 4 + 128) * (1024 / NT) <= 163840, "four waves per SIMD");
};

// Image index -> lower node and upper weight along one axis, for a ratio of 2
// or 4: voxel i = q R + k lies at node coordinate q + (2k+1)/(2R).
template <int R>
__device__ inline int node_of(int i) {
    return i / R;
}
template <int R>
__device__ inline float w1_of(int i) {
    return static_cast<float>(2 * (i % R) + 1) * (0.5f / R);
}
// the same of a uniform index, by scalar selection
template <int R>
__device__ inline double w1_uniform(int i) {
    if constexpr (R == 2)
        return (i & 1) ? 0.75 : 0.25;
    else
        return (i & 2) ? ((i & 1) ? 0.875 : 0.625) : ((i & 1) ? 0.375 : 0.125);
}

// Halo position s (< NRING) in the two-voxel box: the faces of the one-voxel
// halo (y faces, then z faces), the faces of the two-voxel halo, then the four
// corners of the one-voxel halo.
template <int TY, int TZ>
__device__ inline void ring_pos(int s, int& by, int& bz) {
    using L = March<TY, TZ, 2>;
    const bool outer = s >= L::NFACE;
    const int o = outer ? s - L::NFACE : s;
    const int e = outer ? 1 : 0;
    if (o < 2 * TZ) {
        by = o < TZ ? 1 - e : TY + 2 + e;
        bz = 2 + o % TZ;
    } else if (o < L::NFACE) {
        const int q = o - 2 * TZ;
        by = 2 + (q >> 1);
        bz = (q & 1) ? TZ + 2 + e : 1 - e;
    } else {
        const int q = o - L::NFACE;
        by = (q & 1) ? TY + 2 : 1;
        bz = (q & 2) ? TZ + 2 : 1;
    }
}

// A value that is the same in every lane, in a scalar register.
__device__ inline float uniform(float v) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// Fixes where v is computed: without it the compiler sinks what forms dT into
// the stage that uses it two planes later and carries its many operands over.
__device__ inline void settle(float& v) { asm volatile("" : "+v"(v)); }

__device__ inline bool settle_and(bool u, bool v) {
    uint64_t m = __builtin_amdgcn_ballot_w64(u) & __builtin_amdgcn_ballot_w64(v);
    asm volatile("" : "+s"(m));
    return __builtin_amdgcn_inverse_ballot_w64(m);
}

template <int CTRL>
__device__ inline float dpp(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}

// Sum along z of a node cell's voxels (neighbouring lanes), weighted for the
// cell's lower node on the first lane of the cell and for its upper node on
// the second.
template <int R>
__device__ inline float cell_sum_z(float v, float w0, float w1) {
    if constexpr (R == 2) {
        // lane 0: 3/4 own + 1/4 other; lane 1, for the upper node: the same
        return fmaf(0.25f, dpp<0xB1>(v), 0.75f * v);
    } else {
        float lo = w0 * v, hi = w1 * v;
        lo += dpp<0xB1>(lo);
        lo += dpp<0x4E>(lo);
        hi += dpp<0xB1>(hi);
        hi += dpp<0x4E>(hi);
        return (threadIdx.x & 1) ? hi : lo;
    }
}

// SENS: e is also stored, for the template gradient
template <int TY, int TZ, int R, bool GRAD, bool POW2, bool SENS = false>
__device__ __forceinline__ void march_body(const ImagePassArgs& a, int CX, int block) {
    using L = March<TY, TZ, R>;
    constexpr int NT = L::NT, H2Z = L::H2Z;
    constexpr int LEAD = GRAD ? 2 : 1;  // planes before (and after) the chunk a stencil reads
    extern __shared__ float smem[];
    double* sQ = reinterpret_cast<double*>(smem);
    float* sTy = smem + L::OFF_TY;
    float* sR = smem + L::OFF_R;
    float* sVy = smem + L::OFF_VY;
    float* sVz = smem + L::OFF_VZ;
    float* sG = smem + L::OFF_G;
    __shared__ double red[NT / 64];

    // tile decode, spread over the XCDs so that neighbouring tiles share an L2
    const int t = threadIdx.x;
    const int tile = xcd_tile(block, a.ntx * a.nty * a.ntz);
    const int tz = tile % a.ntz;
    const int ty = (tile / a.ntz) % a.nty;
    const int tx = tile / (a.ntz * a.nty);
    const int x0 = tx * CX, y0 = ty * TY, z0 = tz * TZ;
    const int mx = a.mx, my = a.my, mz = a.mz;
    const int sxT = my * mz;
    const int nnod = a.nx * a.ny * a.nz;
    const int qly = max(y0 - 2, 0) / R, qlz = max(z0 - 2, 0) / R;
    const int xend = min(x0 + CX, mx);  // first plane past the chunk (in the domain)
    const uint32_t plane4 = static_cast<uint32_t>(sxT) * 4u, row4 = static_cast<uint32_t>(mz) * 4u;
    const uint32_t nplane4 = static_cast<uint32_t>(a.ny * a.nz) * 4u;
    const __amdgpu_buffer_rsrc_t rT = make_rsrc(a.T, static_cast<uint32_t>(mx) * plane4);
    const __amdgpu_buffer_rsrc_t rR = make_rsrc(a.R, static_cast<uint32_t>(mx) * plane4);
    const __amdgpu_buffer_rsrc_t rY = make_rsrc(a.y, 3u * static_cast<uint32_t>(nnod) * 4u);

    // uniform operands, in scalar registers
    const float tau2 = uniform(a.tau * a.tau), rho2 = uniform(a.rho * a.rho);
    const float taurho = uniform(a.tau * a.rho), nhbar = uniform(-a.hbar);

    // ---- this thread's positions: tile voxels A and B, halo position C ----
    // A and B.  Where the tile ends outside the domain (ragged), threads there
    // compute values nobody reads and write nothing; the last rows and columns
    // inside write the replicated ghosts beside them.
    const int lz = t % TZ, ly = 2 * (t / TZ);
    const bool ragged = y0 + TY > my || z0 + TZ > mz;
    const bool inside = y0 + ly < my && z0 + lz < mz;  // both rows, or neither
    const bool row_end = ragged && inside && y0 + ly + 2 == my && ly + 2 < TY;
    const bool col_end = ragged && inside && z0 + lz + 1 == mz && lz + 1 < TZ;
    const int box = (ly + 2) * H2Z + lz + 2;  // place of A in the two-voxel box, B a row on
    const uint32_t offA = static_cast<uint32_t>(min(y0 + ly, my - 1) * mz + min(z0 + lz, mz - 1)) * 4u;
    const int qA = 3 * (((y0 + min(ly, my - 1 - y0)) / R - qly) * L::NQZ +
                        ((z0 + min(lz, mz - 1 - z0)) / R - qlz));
    const float wyA = R == 2 ? 0.25f : ((ly & 2) ? 0.625f : 0.125f), wyB = wyA + 1.0f / R;
    const float wz = w1_of<R>(lz);
    double dwA = wyA, dwB = wyB;
    if (R == 2) asm volatile("" : "+s"(dwA), "+s"(dwB));
    // C, clamped into the domain (the value of a ghost is its voxel's): its
    // place in the box and its voxel's, its image offset, Q offset and weights
    // and the slot its v_y or v_z goes to
    int byC, bzC;
    ring_pos<TY, TZ>(min(t, L::NRING - 1), byC, bzC);
    const int cyC = clampi(y0 - 2 + byC, 0, my - 1), czC = clampi(z0 - 2 + bzC, 0, mz - 1);
    const uint32_t offC = static_cast<uint32_t>(cyC * mz + czC) * 4u;
    float wyC = w1_of<R>(cyC), wzC = w1_of<R>(czC);
    const bool face = t < L::NFACE, yface = t < 2 * TZ;
    const bool flipC = yface ? cyC != y0 - 2 + byC : czC != z0 - 2 + bzC;
    uint32_t packC1 = static_cast<uint32_t>(byC * H2Z + bzC) |
                      static_cast<uint32_t>((cyC - y0 + 2) * H2Z + (czC - z0 + 2)) << 16;
    uint32_t packC2 = static_cast<uint32_t>(3 * ((cyC / R - qly) * L::NQZ + (czC / R - qlz))) |
                      static_cast<uint32_t>(yface ? (byC - 1) * TZ + (bzC - 2)
                                                  : (byC - 2) * (TZ + 2) + (bzC - 1))
                          << 16;

    // ---- node plane of P: x-interpolated nodes of one image plane ----------
    uint32_t qo[L::KQ];
#pragma unroll
    for (int k = 0; k < L::KQ; ++k) {
        const int i = min(t + k * NT, 3 * L::NQ - 1);
        const int r = i / 3, c = i - 3 * r;
        const int gy = min(qly + r / L::NQZ, a.ny - 1), gz = min(qlz + r % L::NQZ, a.nz - 1);
        qo[k] = static_cast<uint32_t>(c * nnod + gy * a.nz + gz) * 4u;
    }
    auto load_q = [&](int p, float (&q0)[L::KQ], float (&q1)[L::KQ]) {
        const uint32_t j = static_cast<uint32_t>(node_of<R>(clampi(p, 0, mx - 1))) * nplane4;
#pragma unroll
        for (int k = 0; k < L::KQ; ++k) {
            q0[k] = bload(rY, qo[k], j);
            q1[k] = bload(rY, qo[k], j + nplane4);
        }
    };
    auto store_q = [&](int p, int slot, const float (&q0)[L::KQ], const float (&q1)[L::KQ]) {
        const int pc = clampi(p, 0, mx - 1);
        const double w1 = w1_uniform<R>(pc), w0 = w1_uniform<R>(~pc);  // mirrored within the cell: 1 - w1
        double* Q = sQ + slot * 3 * L::NQ;
#pragma unroll
        for (int k = 0; k < L::KQ; ++k)
            if ((k + 1) * NT <= 3 * L::NQ || t + k * NT < 3 * L::NQ)
                Q[t + k * NT] = w0 * static_cast<double>(q0[k]) + w1 * static_cast<double>(q1[k]);
    };

    // y_hat of a position from its four nodes of plane Q: along z, then y
    auto lerp_z = [&](const double* Q, double w, double& lo, double& up) {
        lo = fma(w, Q[3] - Q[0], Q[0]);
        up = fma(w, Q[3 * L::NQZ + 3] - Q[3 * L::NQZ], Q[3 * L::NQZ]);
    };
    // Cell and fraction of the template index, clamped into the domain; in:
    // inside it.  The cell is in [0, m - 2], so the fraction reaches 1 at the
    // far end and lies outside [0, 1] exactly where the index is outside (a
    // NaN counts as outside, with cell and fraction 0).
    auto cell_of = [&](const double (&yh)[3], float (&f)[3], bool (&in)[3],
                       bool slope) -> uint32_t {
        const double hh[3] = {a.hx, a.hy, a.hz}, ih[3] = {a.ihx, a.ihy, a.ihz};
        const int last[3] = {mx - 2, my - 2, mz - 2};
        int i0[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double xi = index_of<POW2>(yh[d], hh[d], ih[d]);
            i0[d] = min(max(to_int(xi), 0), last[d]);
            const double r = xi - static_cast<double>(i0[d]);
            f[d] = __builtin_amdgcn_fmed3f(static_cast<float>(r), 0.0f, 1.0f);
            settle(f[d]);
            if (GRAD && slope) in[d] = settle_and(r >= 0.0, r <= 1.0);
        }
        return static_cast<uint32_t>((i0[0] * my + i0[1]) * mz + i0[2]) * 4u;
    };
    auto gather = [&](uint32_t tb, float2 (&v)[4]) {
        v[0] = bload2(rT, tb, 0u);
        v[1] = bload2(rT, tb, row4);
        v[2] = bload2(rT, tb, plane4);
        v[3] = bload2(rT, tb, plane4 + row4);
    };
    auto interp = [&](const float2 (&v)[4], const float (&f)[3], const bool (&in)[3],
                      float* dT) -> float {
        const float qx = 1.0f - f[0], qy = 1.0f - f[1], qz = 1.0f - f[2];
        const float c00 = fmaf(f[2], v[0].y, qz * v[0].x), c01 = fmaf(f[2], v[1].y, qz * v[1].x);
        const float c10 = fmaf(f[2], v[2].y, qz * v[2].x), c11 = fmaf(f[2], v[3].y, qz * v[3].x);
        const float c0 = fmaf(f[1], c01, qy * c00), c1 = fmaf(f[1], c11, qy * c10);
        if (GRAD && dT != nullptr) {
            const float d0 = c01 - c00, d1 = c11 - c10;
            const float e00 = v[0].y - v[0].x, e01 = v[1].y - v[1].x;
            const float e10 = v[2].y - v[2].x, e11 = v[3].y - v[3].x;
            const float ez0 = fmaf(f[1], e01, qy * e00), ez1 = fmaf(f[1], e11, qy * e10);
            dT[0] = in[0] ? (c1 - c0) * a.fihx : 0.0f;
            dT[1] = in[1] ? fmaf(f[0], d1, qx * d0) * a.fihy : 0.0f;
            dT[2] = in[2] ? fmaf(f[0], ez1, qx * ez0) * a.fihz : 0.0f;
        }
        return fmaf(f[0], c1, qx * c0);
    };

    // ---- rolling state, plane p of a step in slot (step mod 3) --------------
    float tA[3] = {0, 0, 0}, tB[3] = {0, 0, 0}, tC[3] = {0, 0, 0};  // T_y at A, B, C
    float rA[3] = {0, 0, 0}, rB[3] = {0, 0, 0}, rC[3] = {0, 0, 0};  // R at A, B, C
    float dA[3][3] = {}, dB[3][3] = {};                             // dT_y/dy_hat at A, B
    float xA[3] = {0, 0, 0}, xB[3] = {0, 0, 0};                     // v_x at A, B
    float acc0[6] = {}, acc1[6] = {};  // P^T of node planes jA, jA+1: [c][lower, upper y node]
    int jA = x0 / R, pend = -1;
    double dsum = 0.0;
    const int NPc = (CX / R + 1) * L::PY * L::PZ;
    float* part = a.part + static_cast<int64_t>(tile) * 3 * NPc;

    // completed node plane: its z sums to LDS; one barrier later the y sums
    // over neighbouring pairs and the store
    auto stage = [&](const float (&acc)[6]) {
#pragma unroll
        for (int i = 0; i < 6; ++i) sG[i * NT + t] = cell_sum_z<R>(acc[i], 1.0f - wz, wz);
    };
    auto emit = [&](int lx) {
        // one node a thread, its three components; the last waves (the first
        // ones have the halo)
        int i = t - (NT - L::PY * L::PZ);
        asm volatile("" : "+v"(i));  // its places are worked out here, not kept over the loop
        if (i < 0) return;
        const int ny = i / L::PZ, nz = i - ny * L::PZ;
        // the node's cells below (their upper node) and above, along y and z
        const bool yb = ny > 0, ya = ny < L::BY, zb = nz > 0, za = nz < L::BZ;
        const float* gb = sG + NT + max(ny - 1, 0) * (R / 2) * TZ;
        const float* ga = sG + min(ny, L::BY - 1) * (R / 2) * TZ;
        const int ob = max(nz - 1, 0) * R + 1, oa = min(nz, L::BZ - 1) * R;
        float* out = part + lx * (L::PY * L::PZ) + i;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            float v = 0.0f;
#pragma unroll
            for (int p = 0; p < R / 2; ++p) {
                v += yb && zb ? gb[2 * c * NT + p * TZ + ob] : 0.0f;
                v += yb && za ? gb[2 * c * NT + p * TZ + oa] : 0.0f;
                v += ya && zb ? ga[2 * c * NT + p * TZ + ob] : 0.0f;
                v += ya && za ? ga[2 * c * NT + p * TZ + oa] : 0.0f;
            }
            out[c * NPc] = v;
        }
    };

    {
        float q0[L::KQ], q1[L::KQ];
        load_q(x0 - LEAD, q0, q1);
        store_q(x0 - LEAD, 0, q0, q1);
    }
    __syncthreads();

    const int nstep = xend - x0 + 2 * LEAD;
    // One step: plane pw = x0 - LEAD + k enters.  Whatever it reads from LDS
    // was written in an earlier step.
    auto step = [&](auto slot, const int k) {
        constexpr int S = decltype(slot)::value;
        constexpr int S0 = S % 3, S1 = (S + 2) % 3, S2 = (S + 1) % 3;
        constexpr int P0 = S & 1, P1 = P0 ^ 1;  // LDS slots written in this step, in the last one
        const int pw = x0 - LEAD + k;
        const uint32_t pwc4 = static_cast<uint32_t>(clampi(pw, 0, mx - 1)) * plane4;
        // halo positions this plane needs: all of them where v is formed on
        // the halo's faces, the faces beside those planes, none at the ends
        const bool mid = pw >= x0 && pw < xend;
        const bool edge = GRAD && (pw == x0 - 1 || pw == xend);
        const int nring = mid ? (GRAD ? L::NRING : L::NFACE) : (edge ? L::NFACE : 0);
        const bool ring = t < nring;
        // unpacked and widened where used, not kept so over the loop
        asm volatile("" : "+v"(packC1), "+v"(packC2), "+v"(wyC), "+v"(wzC));
        // ------------- W: P and the warp of plane pw ------------------------
        float2 vC[4];
        float fC[3];
        const double* Q = sQ + P0 * 3 * L::NQ;
        {
            rA[S0] = bload(rR, offA, pwc4);
            rB[S0] = bload(rR, offA, pwc4 + row4);
            if (ring) rC[S0] = bload(rR, offC, pwc4);
            float2 vA[4], vB[4];
            float fA[3], fB[3];
            bool iA[3], iB[3];
            {
                double yA[3], yB[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    double lo, up;
                    lerp_z(Q + qA + c, wz, lo, up);
                    const double d = up - lo;
                    yA[c] = fma(dwA, d, lo);
                    yB[c] = fma(dwB, d, lo);
                }
                gather(cell_of(yA, fA, iA, true), vA);
                gather(cell_of(yB, fB, iB, true), vB);
            }
            tA[S0] = interp(vA, fA, iA, dA[S0]);
            tB[S0] = interp(vB, fB, iB, dB[S0]);
            if (GRAD) {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    settle(dA[S0][c]);
                    settle(dB[S0][c]);
                }
            }
        }
        if (ring) {
            const int qC = packC2 & 0xffffu;
            double yC[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                double lo, up;
                lerp_z(Q + qC + c, wzC, lo, up);
                yC[c] = fma(static_cast<double>(wyC), up - lo, lo);
            }
            bool iC[3];
            gather(cell_of(yC, fC, iC, false), vC);
        }
        float q0[L::KQ], q1[L::KQ];  // nodes of the next plane, stored at the end of the step
        if (k + 1 < nstep) load_q(pw + 1, q0, q1);
        // ------------- V: NGF on plane pv = pw - 1 --------------------------
        const int pv = pw - 1;
        const bool vin = pv >= x0 && pv < xend;
        const float* T0 = sTy + P1 * L::NH2;
        const float* R0 = sR + P1 * L::NH2;
        // NGF term at one position from its central differences (doubled)
        auto ngf = [&](float Tx, float Ty, float Tz, float Rx, float Ry, float Rz, bool val,
                       float& vx, float& vy, float& vz) {
            const float gTx = Tx * a.i2hx, gTy = Ty * a.i2hy, gTz = Tz * a.i2hz;
            const float gRx = Rx * a.i2hx, gRy = Ry * a.i2hy, gRz = Rz * a.i2hz;
            const float aa = fmaf(gTx, gTx, fmaf(gTy, gTy, fmaf(gTz, gTz, tau2)));
            const float bb = fmaf(gRx, gRx, fmaf(gRy, gRy, fmaf(gRz, gRz, rho2)));
            const float ab = fmaf(gTx, gRx, fmaf(gTy, gRy, fmaf(gTz, gRz, taurho)));
            const float iaa = __builtin_amdgcn_rcpf(aa), ibb = __builtin_amdgcn_rcpf(bb);
            if (val) {
                // 1 - r^2 = (aa bb - ab^2) / (aa bb) with a = (grad T, tau), b = (grad R,
                // rho), products unfused: exactly 0 when a = b (aa = bb = ab bit for bit)
                float lag;
                {
#pragma clang fp contract(off)
                    lag = aa * bb - ab * ab;
                }
                const float term = lag * iaa * ibb;
                dsum += static_cast<double>(inside ? term : 0.0f);
            }
            if (GRAD) {
                // v = -hbar r/(nT nR) (grad R - (c/nT^2) grad T)
                //   = -hbar ab/(aa^2 bb) (aa grad R - ab grad T),
                // with unfused products so that v is exactly 0 when grad T = grad R
                // (then ab = aa bit for bit and both products round alike)
                const float coef = nhbar * ab * (iaa * iaa) * ibb;
                float wx, wy, wzz;
                {
#pragma clang fp contract(off)
                    wx = aa * gRx - ab * gTx;
                    wy = aa * gRy - ab * gTy;
                    wzz = aa * gRz - ab * gTz;
                }
                vx = coef * wx;
                vy = coef * wy;
                vz = coef * wzz;
            }
        };
        if (vin || (GRAD && pv >= max(x0 - 1, 0) && pv <= min(xend, mx - 1))) {
            const float* TA = T0 + box;
            const float* RA = R0 + box;
            float* Vy = sVy + P0 * L::VYS + (ly + 1) * TZ + lz;
            float* Vz = sVz + P0 * L::VZS + ly * (TZ + 2) + lz + 1;
            float vy, vz;
            ngf(tA[S0] - tA[S2], tB[S1] - TA[-H2Z], TA[1] - TA[-1], rA[S0] - rA[S2],
                rB[S1] - RA[-H2Z], RA[1] - RA[-1], vin, xA[S0], vy, vz);
            if (GRAD && vin && (!ragged || inside)) {
                Vy[0] = vy;
                Vz[0] = vz;
                if (col_end) Vz[1] = -vz;  // mirrored ghosts of the y and z adjoint stencils
            }
            ngf(tB[S0] - tB[S2], TA[2 * H2Z] - tA[S1], TA[H2Z + 1] - TA[H2Z - 1], rB[S0] - rB[S2],
                RA[2 * H2Z] - rA[S1], RA[H2Z + 1] - RA[H2Z - 1], vin, xB[S0], vy, vz);
            if (GRAD && vin) {
                if (!ragged || inside) {
                    Vy[TZ] = vy;
                    Vz[TZ + 2] = vz;
                    if (col_end) Vz[TZ + 3] = -vz;
                    if (row_end) Vy[2 * TZ] = -vy;
                }
            }
        }
        // the halo position: its gathers were in flight over the tile's V
        if (ring) {
            const bool none[3] = {false, false, false};
            tC[S0] = interp(vC, fC, none, nullptr);
        }
        if (GRAD && vin && face) {
            const float* TC = T0 + (packC1 >> 16);
            const float* RC = R0 + (packC1 >> 16);
            float vx, vy, vz;
            ngf(tC[S0] - tC[S2], TC[H2Z] - TC[-H2Z], TC[1] - TC[-1], rC[S0] - rC[S2],
                RC[H2Z] - RC[-H2Z], RC[1] - RC[-1], false, vx, vy, vz);
            const float v = yface ? vy : vz;
            (yface ? sVy + P0 * L::VYS : sVz + P0 * L::VZS)[packC2 >> 16] = flipC ? -v : v;
        }
        if (GRAD) {
            if (pend >= 0) {
                emit(pend);
                pend = -1;
            }
            // ------------- E: adjoint on plane pe = pw - 2, P^T along y and x ---
            const int pe = pw - 2;
            if (pe >= x0) {
                const int jx = node_of<R>(pe);
                const float wx1 = static_cast<float>(w1_uniform<R>(pe));
                const float wx0 = static_cast<float>(w1_uniform<R>(~pe));
                if (jx > jA) {  // node plane jA has all its image planes
                    stage(acc0);
                    pend = jA - x0 / R;
#pragma unroll
                    for (int i = 0; i < 6; ++i) {
                        acc0[i] = acc1[i];
                        acc1[i] = 0.0f;
                    }
                    jA += 1;
                }
                const float* Vy = sVy + P1 * L::VYS + ly * TZ + lz;
                const float* Vz = sVz + P1 * L::VZS + ly * (TZ + 2) + lz;
                // mirrored ghosts of the x adjoint stencil at the domain's ends
                const bool lo = pe > 0, up = pe + 1 < mx;
                const float exA = (lo ? xA[S2] : -xA[S1]) - (up ? xA[S0] : -xA[S1]);
                const float exB = (lo ? xB[S2] : -xB[S1]) - (up ? xB[S0] : -xB[S1]);
                const float eyA = Vy[0] - Vy[2 * TZ], eyB = Vy[TZ] - Vy[3 * TZ];
                const float ezA = Vz[0] - Vz[2], ezB = Vz[TZ + 2] - Vz[TZ + 4];
                float eA = fmaf(exA, a.i2hx, fmaf(eyA, a.i2hy, ezA * a.i2hz));
                float eB = fmaf(exB, a.i2hx, fmaf(eyB, a.i2hy, ezB * a.i2hz));
                if (ragged) {
                    eA = inside ? eA : 0.0f;
                    eB = inside ? eB : 0.0f;
                }
                if (SENS && inside) {
                    const __amdgpu_buffer_rsrc_t rS =
                        make_rsrc(a.sens, static_cast<uint32_t>(mx) * plane4);
                    const uint32_t pe4 = static_cast<uint32_t>(pe) * plane4;
                    bstore(rS, eA, offA, pe4);
                    bstore(rS, eB, offA, pe4 + row4);
                }
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const float gA = eA * dA[S2][c], gB = eB * dB[S2][c];
                    const float gl = fmaf(1.0f - wyB, gB, (1.0f - wyA) * gA);
                    const float gu = fmaf(wyB, gB, wyA * gA);
                    acc0[2 * c] = fmaf(wx0, gl, acc0[2 * c]);
                    acc0[2 * c + 1] = fmaf(wx0, gu, acc0[2 * c + 1]);
                    acc1[2 * c] = fmaf(wx1, gl, acc1[2 * c]);
                    acc1[2 * c + 1] = fmaf(wx1, gu, acc1[2 * c + 1]);
                }
            }
        }
        // ------------- what the next step reads -------------------------------
        float* Tw = sTy + P0 * L::NH2 + box;
        float* Rw = sR + P0 * L::NH2 + box;
        if (!ragged || inside) {
            Tw[0] = tA[S0];
            Tw[H2Z] = tB[S0];
            Rw[0] = rA[S0];
            Rw[H2Z] = rB[S0];
            if (row_end) {
                Tw[2 * H2Z] = tB[S0];
                Rw[2 * H2Z] = rB[S0];
            }
            if (col_end) {
                Tw[1] = tA[S0];
                Tw[H2Z + 1] = tB[S0];
                Rw[1] = rA[S0];
                Rw[H2Z + 1] = rB[S0];
            }
        }
        if (ring) {
            const int bc = packC1 & 0xffffu;
            sTy[P0 * L::NH2 + bc] = tC[S0];
            sR[P0 * L::NH2 + bc] = rC[S0];
        }
        if (k + 1 < nstep) store_q(pw + 1, P1, q0, q1);
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
    if (GRAD) {
        if (pend >= 0) emit(pend);
        __syncthreads();
        stage(acc0);
        __syncthreads();
        emit(jA - x0 / R);
        __syncthreads();
        stage(acc1);
        __syncthreads();
        emit(jA + 1 - x0 / R);
    }
    // D partial of the tile: wave sums, then the waves in order
    const double v = wave_sum(dsum);
    if ((t & 63) == 0) red[t >> 6] = v;
    __syncthreads();
    if (t == 0) {
        double s = (red[0] + red[1]) + (red[2] + red[3]);
        if constexpr (NT == 512) s += (red[4] + red[5]) + (red[6] + red[7]);
        a.dpart[tile] = s;
    }
}

template <int TY, int TZ, int R, bool GRAD, bool POW2>
__global__ __launch_bounds__((March<TY, TZ, R>::NT), 4) void k_image_march(
    ImagePassArgs a, int CX) {
    if (a.gate && *a.gate == kOpNone) return;
    march_body<TY, TZ, R, GRAD, POW2>(a, CX, blockIdx.x);
}

template <int TY, int TZ, int R, bool POW2>
__global__ __launch_bounds__((March<TY, TZ, R>::NT), 4) void k_image_march_sens(
    ImagePassArgs a, int CX) {
    march_body<TY, TZ, R, true, POW2, true>(a, CX, blockIdx.x);
}

// Each pair's chunk length is its own (a.cx).  The pair and block indices
// are uniform over the workgroup: taken as such, the pair's arguments load
// into scalar registers and the kernel needs no more vector registers than
// the single-pair one (no spills).
template <int TY, int TZ, int R, bool POW2>
__global__ __launch_bounds__((March<TY, TZ, R>::NT), 4) void k_image_march_batch(
    const ImagePassArgs* args, const BlockRef* blk) {
    const BlockRef e = blk[blockIdx.x];
    const int pair = __builtin_amdgcn_readfirstlane(e.pair);
    if (pair < 0) return;
    const ImagePassArgs a = args[pair];
    if (a.gate && *a.gate == kOpNone) return;
    march_body<TY, TZ, R, true, POW2>(a, __builtin_amdgcn_readfirstlane(a.cx),
                                      __builtin_amdgcn_readfirstlane(e.block));
}

template <int TY, int TZ, int R>
void launch_march_batch_t(const ImagePassArgs* args, const BlockRef* blk, int nblk, bool pow2,
                          hipStream_t s) {
    using L = March<TY, TZ, R>;
    const size_t lds = sizeof(float) * L::LDS_GRAD;
    if (pow2)
        hipLaunchKernelGGL((k_image_march_batch<TY, TZ, R, true>), dim3(nblk), dim3(L::NT),
                           lds, s, args, blk);
    else
        hipLaunchKernelGGL((k_image_march_batch<TY, TZ, R, false>), dim3(nblk), dim3(L::NT),
                           lds, s, args, blk);
}

template <int TY, int TZ, int R>
void launch_march_t(const ImagePassArgs& a, int cx, hipStream_t s) {
    using L = March<TY, TZ, R>;
    const int blocks = a.ntx * a.nty * a.ntz;
    const size_t lds = sizeof(float) * (a.want_grad ? L::LDS_GRAD : L::LDS_VALUE);
    // the spacing decides at compile time how the warp index is formed
    if (a.want_grad) {
        if (a.pow2h)
            hipLaunchKernelGGL((k_image_march<TY, TZ, R, true, true>), dim3(blocks),
                               dim3(L::NT), lds, s, a, cx);
        else
            hipLaunchKernelGGL((k_image_march<TY, TZ, R, true, false>), dim3(blocks),
                               dim3(L::NT), lds, s, a, cx);
    } else {
        if (a.pow2h)
            hipLaunchKernelGGL((k_image_march<TY, TZ, R, false, true>), dim3(blocks),
                               dim3(L::NT), lds, s, a, cx);
        else
            hipLaunchKernelGGL((k_image_march<TY, TZ, R, false, false>), dim3(blocks),
                               dim3(L::NT), lds, s, a, cx);
    }
}

template <int TY, int TZ, int R>
void launch_march_sens_t(const ImagePassArgs& a, int cx, hipStream_t s) {
    using L = March<TY, TZ, R>;
    const dim3 g(a.ntx * a.nty * a.ntz), b(L::NT);
    const size_t lds = sizeof(float) * L::LDS_GRAD;
    if (a.pow2h)
        hipLaunchKernelGGL((k_image_march_sens<TY, TZ, R, true>), g, b, lds, s, a, cx);
    else
        hipLaunchKernelGGL((k_image_march_sens<TY, TZ, R, false>), g, b, lds, s, a, cx);
}

}  // namespace

void launch_image_march_sens(const ImagePassArgs& a, int ratio, int ty, int cx, hipStream_t s) {
    if (ty == 32) {
        if (ratio == 2)
            launch_march_sens_t<32, 32, 2>(a, cx, s);
        else
            launch_march_sens_t<32, 32, 4>(a, cx, s);
    } else {
        if (ratio == 2)
            launch_march_sens_t<kMY, 32, 2>(a, cx, s);
        else
            launch_march_sens_t<kMY, 32, 4>(a, cx, s);
    }
}

// gradient form only (the batched rounds always want the gradient)
void launch_image_march_batch(const ImagePassArgs* args, const BlockRef* blk, int nblk,
                              int ratio, int variant, bool pow2, hipStream_t s) {
    if (nblk <= 0) return;
    const int ty = march_ty(variant), tz = march_tz(variant);
    if (ty == 32) {
        if (ratio == 2)
            launch_march_batch_t<32, 32, 2>(args, blk, nblk, pow2, s);
        else if (ratio == 4)
            launch_march_batch_t<32, 32, 4>(args, blk, nblk, pow2, s);
    } else if (tz == 64) {
        if (ratio == 2)
            launch_march_batch_t<kMY, 64, 2>(args, blk, nblk, pow2, s);
        else if (ratio == 4)
            launch_march_batch_t<kMY, 64, 4>(args, blk, nblk, pow2, s);
    } else {
        if (ratio == 2)
            launch_march_batch_t<kMY, 32, 2>(args, blk, nblk, pow2, s);
        else if (ratio == 4)
            launch_march_batch_t<kMY, 32, 4>(args, blk, nblk, pow2, s);
    }
}

namespace {
template <int TY, int TZ>
int march_per_cu() {
    using L = March<TY, TZ, 2>;
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_image_march<TY, TZ, 2, true, true>,
                                                     L::NT, sizeof(float) * L::LDS_GRAD) !=
            hipSuccess ||
        per_cu < 1)
        per_cu = 1;
    return per_cu;
}
}  // namespace

int image_march_slots(int ty, int tz) {
    // occupancy per CU, queried once per device and tile (the ratio-2
    // instance stands for both ratios: its LDS is the larger, and either has
    // four waves per SIMD)
    static std::atomic<int> cache[16][3];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) dev = 0;
    const int form = ty == 32 ? 2 : (tz == 64 ? 1 : 0);
    std::atomic<int>& slot = cache[dev & 15][form];
    int v = slot.load();
    if (v > 0) return v;
    const int per_cu = form == 2 ? march_per_cu<32, 32>()
                                 : (form == 1 ? march_per_cu<kMY, 64>() : march_per_cu<kMY, 32>());
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus < 1)
        cus = 256;
    (void)hipGetLastError();
    v = per_cu * cus;
    slot.store(v);
    return v;
}

void launch_image_march(const ImagePassArgs& a, int ratio, int ty, int tz, int cx,
                        hipStream_t s) {
    if (ty == 32) {
        if (ratio == 2)
            launch_march_t<32, 32, 2>(a, cx, s);
        else if (ratio == 4)
            launch_march_t<32, 32, 4>(a, cx, s);
    } else if (tz == 64) {
        if (ratio == 2)
            launch_march_t<kMY, 64, 2>(a, cx, s);
        else if (ratio == 4)
            launch_march_t<kMY, 64, 4>(a, cx, s);
    } else {
        if (ratio == 2)
            launch_march_t<kMY, 32, 2>(a, cx, s);
        else if (ratio == 4)
            launch_march_t<kMY, 32, 4>(a, cx, s);
    }
}

}  // namespace ngf
