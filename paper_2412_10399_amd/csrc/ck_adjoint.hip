// Differentiable compact-kernel MPM step: forward step on dense or block-sparse grids
// and its exact reverse mode (vector-Jacobian product), two lanes per particle, one for
// each grid.
//
// Forward, for particle p at X = (x - origin)/dx (cell units), on grid G_k
// (k = -1 for G-, +1 for G+, node i at i + k/4 cells), per axis a:
//   xi = X_a - k/4 - floor(X_a - k/4), weights of the two nodes
//   w0 = K1(xi) = 1 - xi + s,  w1 = K1(1 - xi) = xi - s,  s = sin(2 pi xi)/(2 pi),
//   dw0/dX = cos(2 pi xi) - 1,  dw1/dX = 1 - cos(2 pi xi)        (section 4.1 kernel);
// w_i is the product over the axes, d_i = x_i - x_p;
//   D = 1/2 sum_k sum_i w d d^T  (section 4.4; per axis the first moment on grid k
//       is -s dx and the second (xi (1 - xi) - s (1 - 2 xi)) dx^2),
//   P2G: m_i += w m,  p_i += w (m v + Q d),  Q = (m B - dt V0 tau) D^-1    (4.3, 4.5),
//   grid: v~ = p/m + dt g where m > 0 and the node is inside the walls, else 0,
//   G2P: v' = 1/2 sum w v~,  B' = 1/2 sum w v~ d^T,  F' = (I + dt B' D^-1) F,
//        x' = x + dt v',
//   tau = 2 mu (F - R) F^T + lambda (J - 1) J I  (fixed corotated), mu and lambda
//   proportional to E = exp(logE).
// Reverse: the three phases in the opposite order, each product rule written out
// next to the line that applies it.
#include "../../include/ckmpm_adjoint.h"
#include "ck_common.hpp"
#include "ck_ctx.hpp"

#include <algorithm>
#include <cmath>
#include <new>

#include <climits>

using namespace ck;

struct mpm_ad_ctx {
    int device = 0;
    Geometry geo;
    float gravity[3];
    float nu, rho, vol0;
    int64_t max_particles = 0;
    int cap = 0;              // pool slots per grid (blocks of 4x4x4 nodes)
    int nb[3] = {0, 0, 0};    // blocks per axis covering the (n+1)^3 node lattice
    long long nbv = 0;        // nb[0] nb[1] nb[2]
    long long nodes = 0;      // nodes of one grid: (n+1)^3 when direct, else (cap + 1) * 64
                              // (pool slots, the last a spill slot)
    float4 *grid = nullptr;   // 3 arrays of 2 * nodes float4, see below
    int *page = nullptr;      // [grid][nbv]: pool slot of a block in this call, -1 if untouched
    bool direct = false;      // max_blocks covers the lattice: dense grids, no marking
    unsigned char *flag = nullptr;   // [grid][nbv]: touched by a particle's stencil
    unsigned int *ctl = nullptr;     // control words, see AdCtl
    unsigned int *status = nullptr;
};

namespace {

// Grids.  When max_blocks covers every 4x4x4-node block of the lattice (`direct`),
// the grids are dense, node (ix, iy, iz) at (iz ny + iy) nx + ix.  Otherwise they are
// block-sparse: each call marks the blocks that its particles' stencils touch
// (k_ad_mark) and gives them pool slots (k_ad_alloc); the node lives at
// page[g][block] * 64 + ((iz & 3) * 4 + (iy & 3)) * 4 + (ix & 3).  Past the pool's
// capacity a block gets the spill slot `cap` (its values meaningless) and the call
// reports ST_CAPACITY.
//
// Arrays of 2 * nodes float4 (G- then G+), a node's values in one 16-byte load:
//   X0, X1  (m, p0, p1, p2): the calls take turns.  P2G sums into one while other
//           workgroups of its launch clear the one that the call before left behind;
//   VB      dL/dv~ (three used): the scatter target of the reverse step, cleared in the
//           same way after a reverse call.
// There is no pass over the grid: G2P and its adjoint form the node velocities
// v~ = p/m + dt g as they gather (m, p), and the P2G adjoint forms the node cotangents
// from (m, p) and dL/dv~.  Which X a call uses is read from the control words, not
// decided on the host, so that a captured sequence of calls can be replayed.
enum AdCtl {
    A_CUR = 0,     // X the next call uses; the call's second kernel writes it (nobody reads it there)
    A_USE = 1,     // X of this call for the kernels after P2G, which writes it
    A_VB = 2,      // VB holds an earlier call's sums; written by the call's second kernel
    A_CNT = 4,     // [2]: slots taken per grid in this call (block-sparse)
    A_PREV = 6,    // [2]: slots taken in the call before
    kCtlWords = 8
};

struct AdArgs {
    Geometry geo;
    float g[3];
    float mass, vol0, nu_mu, nu_lambda;   // mu = nu_mu E, lambda = nu_lambda E
    int nx, ny;   // lattice nodes per axis (direct)
    int nbx, nby, cap;
    long long nbv, nodes;
    float4 *grid;
    int *page;
    int direct;
    unsigned char *flag;
    unsigned int *ctl;
    unsigned int *status;
    int n;
    int pgrid;    // workgroups that take particles, a multiple of 8 (those of P2G past them clear)
    long long stride;
    float dt;
};

__device__ __forceinline__ float4 *ad_x(const AdArgs &a, unsigned int which) {
    return a.grid + ((which & 1u) ? 2 * a.nodes : 0);
}
__device__ __forceinline__ float4 *ad_vb(const AdArgs &a) { return a.grid + 4 * a.nodes; }

// Sets status bits in the context's one status word (read by mpm_ad_sync).
__device__ __forceinline__ void ad_status(const AdArgs &a, unsigned int bits) { atomicOr(a.status, bits); }

// Index of node (ix, iy, iz) of grid g in the node arrays: dense, or in the pool
// (kSparse; the node's block was marked by this call).
template <bool kSparse>
__device__ __forceinline__ long long ad_index(const AdArgs &a, int g, int ix, int iy, int iz) {
    if (!kSparse) return g * a.nodes + ((long long)iz * a.ny + iy) * a.nx + ix;
    const long long b = ((long long)(iz >> 2) * a.nby + (iy >> 2)) * a.nbx + (ix >> 2);
    const int slot = a.page[g * a.nbv + b];
    return g * a.nodes + (long long)slot * 64 + (((iz & 3) * 4 + (iy & 3)) * 4 + (ix & 3));
}

__device__ __forceinline__ bool node_free(const AdArgs &a, int g, int ix, int iy, int iz) {
    return ix >= a.geo.stick_lo[g] && iy >= a.geo.stick_lo[g] && iz >= a.geo.stick_lo[g] &&
           ix <= a.geo.stick_hi[g][0] && iy <= a.geo.stick_hi[g][1] && iz <= a.geo.stick_hi[g][2];
}

// ------------------------------------------------------------ particle stencil
// Two neighbouring lanes share a particle: the even lane takes its stencil on G-, the odd
// one on G+.  A workload of 65,536 particles is one wave per SIMD with a thread per
// particle, bound by each wave's own chain of instructions; the pair halves the chain and
// the registers (the reverse kernels held two grids' stencils in 256 and spilled).  Sums
// over both grids are formed by one exchange within the pair (pair_sum).
struct AdStencil {
    int base[3];        // nodes base + o (o = 0, 1) per axis
    float w[3][2];      // per-axis weights
    float dw[3];        // derivative of w[.][0] with respect to X_a (cell units); w[.][1] has its negative
    float s[3], xi[3];
    float Dinv[9];      // D^-1 in world units (of the particle)
};

__device__ __forceinline__ int pair_grid() { return (int)threadIdx.x & 1; }

// Which 128 particles the workgroup takes.  Workgroups are dealt to the 8 XCDs round-robin
// by index; each XCD gets a contiguous eighth of the particles, so that the nodes which
// neighbouring rows of cells share meet in one L2 (119,223 particles, block-sparse: P2G
// 27.4 -> 26.1 us, G2P adjoint 34.4 -> 33.4 us).
__device__ __forceinline__ int ad_block(const AdArgs &a) {
    return ((int)blockIdx.x & 7) * (a.pgrid >> 3) + ((int)blockIdx.x >> 3);
}

// v of this lane plus v of the pair's other lane (the same value on both).
__device__ __forceinline__ float pair_sum(float v) {
    const int o = __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true);   // quad_perm 1,0,3,2
    return v + __int_as_float(o);
}

// X = (x + r - origin) / dx (the position is x + r, FP32 rounding and remainder,
// summed in FP64); false when the particle is outside the valid domain.
__device__ __forceinline__ bool ad_position(const AdArgs &a, const float x[3], const float r[3], float X[3]) {
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        X[ax] = (float)(((double)x[ax] + (double)r[ax] - a.geo.origin[ax]) * a.geo.inv_dx);
        if (!(X[ax] >= 0.25f && X[ax] < (float)a.geo.n[ax] - 0.25f)) return false;
    }
    return true;
}

// The lane's grid of the particle's stencil; false (and nothing filled in) when the
// particle is outside the valid domain.  Both lanes of a pair call it together.
__device__ __forceinline__ bool ad_stencil(const AdArgs &a, const float x[3], const float r[3], AdStencil &st) {
    constexpr float kInv2Pi = 0.15915494309189535f;
    float X[3];
    if (!ad_position(a, x, r, X)) return false;
    const float k = pair_grid() ? 0.25f : -0.25f;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const float Xk = X[ax] - k;
        const float b = floorf(Xk);
        const float xi = Xk - b;
        st.base[ax] = (int)b;
        const float s = __builtin_amdgcn_sinf(xi) * kInv2Pi;   // argument in revolutions
        st.xi[ax] = xi;
        st.s[ax] = s;
        st.w[ax][0] = 1.0f - xi + s;
        st.w[ax][1] = xi - s;
        st.dw[ax] = __builtin_amdgcn_cosf(xi) - 1.0f;
    }
    // D / dx^2: diagonal 1/2 sum_k (xi (1 - xi) - s (1 - 2 xi)), off-diagonal
    // 1/2 sum_k s_a s_b (the first moments are -s on each grid)
    float Dh[6];   // 00 11 22 01 02 12
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const float xi = st.xi[i];
        Dh[i] = pair_sum(0.5f * (xi * (1.0f - xi) - st.s[i] * (1.0f - 2.0f * xi)));
    }
    Dh[3] = pair_sum(0.5f * st.s[0] * st.s[1]);
    Dh[4] = pair_sum(0.5f * st.s[0] * st.s[2]);
    Dh[5] = pair_sum(0.5f * st.s[1] * st.s[2]);
    // inverse by cofactors (D is symmetric positive definite, condition number < 2)
    const float c00 = Dh[1] * Dh[2] - Dh[5] * Dh[5], c01 = Dh[5] * Dh[4] - Dh[3] * Dh[2],
                c02 = Dh[3] * Dh[5] - Dh[1] * Dh[4];
    const float c11 = Dh[0] * Dh[2] - Dh[4] * Dh[4], c12 = Dh[4] * Dh[3] - Dh[0] * Dh[5];
    const float c22 = Dh[0] * Dh[1] - Dh[3] * Dh[3];
    const float det = Dh[0] * c00 + Dh[3] * c01 + Dh[4] * c02;
    const float sc = a.geo.inv_dx_f * a.geo.inv_dx_f / det;
    st.Dinv[0] = c00 * sc; st.Dinv[1] = c01 * sc; st.Dinv[2] = c02 * sc;
    st.Dinv[3] = c01 * sc; st.Dinv[4] = c11 * sc; st.Dinv[5] = c12 * sc;
    st.Dinv[6] = c02 * sc; st.Dinv[7] = c12 * sc; st.Dinv[8] = c22 * sc;
    return true;
}

// Node o (bits x, y, z; per lane): weight, d = x_i - x_p (world) and the gradient of the
// weight with respect to x_p (world).
__device__ __forceinline__ void ad_weights(const AdArgs &a, const AdStencil &st, int o, float &w, float d[3],
                                           float gw[3]) {
    float wa[3], dwa[3];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const bool up = (o >> ax) & 1;
        wa[ax] = up ? st.w[ax][1] : st.w[ax][0];
        dwa[ax] = (up ? -st.dw[ax] : st.dw[ax]) * a.geo.inv_dx_f;
        d[ax] = ((up ? 1.0f : 0.0f) - st.xi[ax]) * a.geo.dx;
    }
    w = wa[0] * wa[1] * wa[2];
    gw[0] = dwa[0] * wa[1] * wa[2];
    gw[1] = wa[0] * dwa[1] * wa[2];
    gw[2] = wa[0] * wa[1] * dwa[2];
}

// The eight nodes of a stencil are taken from node (particle & 7) on: particles are mostly
// stored cell by cell, eight to a cell, and eight lanes of one cell at the same node
// offset would add to one LDS word eight deep.
__device__ __forceinline__ int ad_turn(int i) { return (i + ((int)threadIdx.x >> 1)) & 7; }

// Whether no node of the lane's stencil lies on a wall (then no node is tested).
__device__ __forceinline__ bool ad_all_free(const AdArgs &a, const AdStencil &st) {
    const int g = pair_grid();
    return node_free(a, g, st.base[0], st.base[1], st.base[2]) &&
           node_free(a, g, st.base[0] + 1, st.base[1] + 1, st.base[2] + 1);
}

// Indices of the eight nodes (node ad_turn(i) in id[i]), and their values in node array
// x, all loads in flight together.
template <bool kSparse>
__device__ __forceinline__ void ad_ids(const AdArgs &a, const AdStencil &st, long long (&id)[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int o = ad_turn(i);
        id[i] = ad_index<kSparse>(a, pair_grid(), st.base[0] + (o & 1), st.base[1] + ((o >> 1) & 1), st.base[2] + (o >> 2));
    }
}
__device__ __forceinline__ void ad_gather(const float4 *x, const long long (&id)[8], float4 (&q)[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) q[i] = x[id[i]];
}

// Grid update of one node: v~ = p/m + dt g where m > 0 and the node is free, else 0.
// Returns 1/m there and 0 elsewhere.
__device__ __forceinline__ float ad_node_velocity(const AdArgs &a, const AdStencil &st, bool all_free, int o,
                                                  const float4 &q, float v[3]) {
    bool live = q.x > 0.0f;
    if (live && !all_free)
        live = node_free(a, pair_grid(), st.base[0] + (o & 1), st.base[1] + ((o >> 1) & 1), st.base[2] + (o >> 2));
    const float im = live ? 1.0f / q.x : 0.0f;
    v[0] = live ? q.y * im + a.dt * a.g[0] : 0.0f;
    v[1] = live ? q.z * im + a.dt * a.g[1] : 0.0f;
    v[2] = live ? q.w * im + a.dt * a.g[2] : 0.0f;
    return im;
}

// Adds to xb the lane's grid's part of the adjoint of D(x_p) for Db = dL/dD (world units):
//   dD/dx_a = dx dD^/dX_a,  dD^_aa/dX_a = 1/2 sum_k ((1 - 2 xi)(1 - c) + 2 s),
//   dD^_ab/dX_a = 1/2 sum_k c_a s_b  (b != a);  other entries do not depend on X_a.
__device__ __forceinline__ void ad_moment_vjp(const AdArgs &a, const AdStencil &st, const float Db[9], float xb[3]) {
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const float c1 = -st.dw[ax];   // 1 - c
        float acc = Db[4 * ax] * 0.5f * ((1.0f - 2.0f * st.xi[ax]) * c1 + 2.0f * st.s[ax]);
#pragma unroll
        for (int b = 0; b < 3; ++b)
            if (b != ax) acc += (Db[3 * ax + b] + Db[3 * b + ax]) * 0.5f * (1.0f - c1) * st.s[b];
        xb[ax] += a.geo.dx * acc;
    }
}

// dL/dD from dL/dD^-1: d(D^-1) = -D^-1 dD D^-1, so Db = -D^-T Dib D^-T (D^-1 symmetric).
__device__ __forceinline__ void ad_inverse_vjp(const float Di[9], const float Dib[9], float Db[9]) {
    float t[9];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) t[3 * i + j] = Dib[3 * i] * Di[j] + Dib[3 * i + 1] * Di[3 + j] + Dib[3 * i + 2] * Di[6 + j];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            Db[3 * i + j] = -(Di[3 * i] * t[j] + Di[3 * i + 1] * t[3 + j] + Di[3 * i + 2] * t[6 + j]);
}

// ------------------------------------------------------------ fixed corotated
// Polar pieces of F = I + H from the eigen-decomposition of F^T F - I (Jacobi):
// V, signed singular values (the smallest negative for an inverted element),
// U = F V diag(1/s), R = U V^T.
struct Polar {
    float U[9], V[9], R[9], s[3];
    float J;
};

__device__ __forceinline__ void ad_polar(const float H[9], Polar &P) {
    Eig3 ev;
    strain_eig(H, ev);
    float W[9];
    mat_W(H, ev.V, W);
    const float J = 1.0f + det_minus_one(H);
    P.J = J;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        float s = fast_sqrt(fmaxf(1.0f + ev.e[i], 1e-30f));
        if (i == 2 && J < 0.0f) s = -s;
        P.s[i] = s;
        const float inv = 1.0f / s;
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            P.U[3 * r + i] = W[3 * r + i] * inv;
            P.V[3 * r + i] = ev.V[3 * r + i];
        }
    }
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            P.R[3 * i + j] = P.U[3 * i] * P.V[3 * j] + P.U[3 * i + 1] * P.V[3 * j + 1] + P.U[3 * i + 2] * P.V[3 * j + 2];
}

// tau = 2 mu (F - R) F^T + lambda (J - 1) J I with (F - R) F^T = W diag((s - 1)/s) W^T,
// W = F V, s - 1 formed from e = s^2 - 1 without cancellation.
__device__ __forceinline__ void ad_tau(const float H[9], const Polar &P, float mu, float lam, float tau[9]) {
    float coef[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const float s = P.s[i];
        const float e = s * s - 1.0f;
        const float sm1 = s > 0.0f ? e / (1.0f + s) : s - 1.0f;
        coef[i] = 2.0f * mu * sm1 / s;
    }
    const float iso = lam * (P.J - 1.0f) * P.J;
    // W_i = s_i U_i
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            float v = (r == c) ? iso : 0.0f;
#pragma unroll
            for (int i = 0; i < 3; ++i) v += coef[i] * P.s[i] * P.s[i] * P.U[3 * r + i] * P.U[3 * c + i];
            tau[3 * r + c] = v;
        }
    (void)H;
}

// Fb += dL/dF for tb = dL/dtau:
//   dtau = 2 mu (dF F^T + F dF^T - dR F^T - R dF^T) + lambda (2J - 1) dJ I,
//   so Fb = 2 mu (tb F + tb^T F - tb^T R) + lambda (2J - 1) tr(tb) cof F, and
//   Rb = -2 mu tb F enters through dR = U M V^T, M_ij = (A_ij - A_ji)/(s_i + s_j),
//   A = U^T dF V:  Fb += U Z V^T,  Z_ij = (Y_ij - Y_ji)/(s_i + s_j),  Y = U^T Rb V.
__device__ __forceinline__ void ad_tau_vjp(const float H[9], const Polar &P, float mu, float lam, const float tb[9],
                                           float Fb[9]) {
    float F[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) F[i] = H[i] + ((i % 4 == 0) ? 1.0f : 0.0f);
    float tF[9], tTF[9], tTR[9];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            float a = 0.0f, b = 0.0f, c = 0.0f;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                a += tb[3 * i + k] * F[3 * k + j];
                b += tb[3 * k + i] * F[3 * k + j];
                c += tb[3 * k + i] * P.R[3 * k + j];
            }
            tF[3 * i + j] = a;
            tTF[3 * i + j] = b;
            tTR[3 * i + j] = c;
        }
    // Y = U^T Rb V with Rb = -2 mu tb F
    float RbV[9], Y[9];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            RbV[3 * i + j] = -2.0f * mu * (tF[3 * i] * P.V[j] + tF[3 * i + 1] * P.V[3 + j] + tF[3 * i + 2] * P.V[6 + j]);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            Y[3 * i + j] = P.U[i] * RbV[j] + P.U[3 + i] * RbV[3 + j] + P.U[6 + i] * RbV[6 + j];
    float Z[9];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) Z[3 * i + j] = (i == j) ? 0.0f : (Y[3 * i + j] - Y[3 * j + i]) / (P.s[i] + P.s[j]);
    // cofactor matrix of F
    float cof[9];
    cof[0] = F[4] * F[8] - F[5] * F[7];
    cof[1] = F[5] * F[6] - F[3] * F[8];
    cof[2] = F[3] * F[7] - F[4] * F[6];
    cof[3] = F[2] * F[7] - F[1] * F[8];
    cof[4] = F[0] * F[8] - F[2] * F[6];
    cof[5] = F[1] * F[6] - F[0] * F[7];
    cof[6] = F[1] * F[5] - F[2] * F[4];
    cof[7] = F[2] * F[3] - F[0] * F[5];
    cof[8] = F[0] * F[4] - F[1] * F[3];
    const float jc = lam * (2.0f * P.J - 1.0f) * (tb[0] + tb[4] + tb[8]);
    // U Z V^T
    float ZV[9];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) ZV[3 * i + j] = Z[3 * i] * P.V[3 * j] + Z[3 * i + 1] * P.V[3 * j + 1] + Z[3 * i + 2] * P.V[3 * j + 2];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const float uzv = P.U[3 * i] * ZV[j] + P.U[3 * i + 1] * ZV[3 + j] + P.U[3 * i + 2] * ZV[6 + j];
            Fb[3 * i + j] += 2.0f * mu * (tF[3 * i + j] + tTF[3 * i + j] - tTR[3 * i + j]) + uzv + jc * cof[3 * i + j];
        }
}

// Coefficients of (1 + x)^(-1/2) - 1 by degree.
__device__ __constant__ const float kInvSqrt[7] = {0.0f,            -0.5f,           0.375f,         -0.3125f,
                                                   35.0f / 128.0f, -63.0f / 256.0f, 231.0f / 1024.0f};

// tau and the adjoint of tau for strains that need no eigen-decomposition (the waves for
// which kirchhoff takes its series): with E = F F^T - I, R = (I + E)^(-1/2) F, so that
// R - I = H + G + G H, G = (I + E)^(-1/2) - I, and F - R = -(G + G H) without
// cancellation.  With F = R S the rotation's derivative is R^T dR = [w]x with
// (tr(S) I - S) w = axial(R^T dF - dF^T R); for Rb = -2 mu tb F that gives
// Fb += R [z]x, (tr(S) I - S) z = axial(Y - Y^T), Y = R^T Rb -- the same map as U Z V^T
// above, without U, V and s.
__device__ __forceinline__ void ad_small_stress(const Sym3 &E, float r2, float jm1, float mu, float lam, float tau[9]) {
    const Sym3 D = power_series(E, kSqrtDiff, wave_terms(r2, kLogThr2, 4, 2));
    const float iso = lam * jm1 * (1.0f + jm1), k = 2.0f * mu;
    tau[0] = k * D.xx + iso; tau[4] = k * D.yy + iso; tau[8] = k * D.zz + iso;
    tau[1] = tau[3] = k * D.xy;
    tau[2] = tau[6] = k * D.xz;
    tau[5] = tau[7] = k * D.yz;
}

// tau of the fixed corotated model, all nine entries; the wave takes the series or the
// eigen-decomposition as kirchhoff does.
__device__ __forceinline__ void ad_stress(const float H[9], float mu, float lam, float tau[9]) {
    const Sym3 E = left_cauchy_green_minus_I(H);
    const float jm1 = det_minus_one(H), r2 = frob2(E);
    if (wave_needs_eig(r2, jm1)) {
        Polar P;
        ad_polar(H, P);
        ad_tau(H, P, mu, lam, tau);
    } else {
        ad_small_stress(E, r2, jm1, mu, lam, tau);
    }
}

__device__ __forceinline__ void mat_mul(const float A[9], const float B[9], float C[9]) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) C[3 * i + j] = A[3 * i] * B[j] + A[3 * i + 1] * B[3 + j] + A[3 * i + 2] * B[6 + j];
}
// A^T B
__device__ __forceinline__ void mat_tmul(const float A[9], const float B[9], float C[9]) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) C[3 * i + j] = A[i] * B[j] + A[3 + i] * B[3 + j] + A[6 + i] * B[6 + j];
}

__device__ __forceinline__ void ad_small_stress_vjp(const float H[9], const Sym3 &E, float r2, float jm1, float mu,
                                                    float lam, const float tb[9], float Fb[9]) {
    const Sym3 G = power_series(E, kInvSqrt, wave_terms(r2, kLogThr2, 4, 2));
    const float g[9] = {G.xx, G.xy, G.xz, G.xy, G.yy, G.yz, G.xz, G.yz, G.zz};
    float F[9], GF[9], R[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) F[i] = H[i] + ((i % 4 == 0) ? 1.0f : 0.0f);
    mat_mul(g, H, GF);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        GF[i] += g[i];           // R - F
        R[i] = F[i] + GF[i];
    }
    float tF[9], tD[9];
    mat_mul(tb, F, tF);
    mat_tmul(tb, GF, tD);        // tb^T (R - F)
    float Y[9], S[9];
    mat_tmul(R, tF, Y);          // Y = -2 mu R^T tb F, the factor below
    mat_tmul(R, F, S);
    const float y0 = Y[7] - Y[5], y1 = Y[2] - Y[6], y2 = Y[3] - Y[1];
    // (tr(S) I - S) z = y: symmetric, eigenvalues s_i + s_j close to two here
    const float m00 = S[4] + S[8], m11 = S[0] + S[8], m22 = S[0] + S[4];
    const float m01 = -0.5f * (S[1] + S[3]), m02 = -0.5f * (S[2] + S[6]), m12 = -0.5f * (S[5] + S[7]);
    const float c00 = m11 * m22 - m12 * m12, c01 = m02 * m12 - m01 * m22, c02 = m01 * m12 - m02 * m11;
    const float c11 = m00 * m22 - m02 * m02, c12 = m01 * m02 - m00 * m12, c22 = m00 * m11 - m01 * m01;
    const float k = -2.0f * mu / (m00 * c00 + m01 * c01 + m02 * c02);
    const float z0 = k * (c00 * y0 + c01 * y1 + c02 * y2), z1 = k * (c01 * y0 + c11 * y1 + c12 * y2),
                z2 = k * (c02 * y0 + c12 * y1 + c22 * y2);
    const float jc = lam * (1.0f + 2.0f * jm1) * (tb[0] + tb[4] + tb[8]);
    float cof[9];
    cof[0] = F[4] * F[8] - F[5] * F[7];
    cof[1] = F[5] * F[6] - F[3] * F[8];
    cof[2] = F[3] * F[7] - F[4] * F[6];
    cof[3] = F[2] * F[7] - F[1] * F[8];
    cof[4] = F[0] * F[8] - F[2] * F[6];
    cof[5] = F[1] * F[6] - F[0] * F[7];
    cof[6] = F[1] * F[5] - F[2] * F[4];
    cof[7] = F[2] * F[3] - F[0] * F[5];
    cof[8] = F[0] * F[4] - F[1] * F[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        // row i of R [z]x
        const float r0 = R[3 * i], r1 = R[3 * i + 1], r2v = R[3 * i + 2];
        const float q[3] = {r1 * z2 - r2v * z1, r2v * z0 - r0 * z2, r0 * z1 - r1 * z0};
#pragma unroll
        for (int j = 0; j < 3; ++j)
            Fb[3 * i + j] += 2.0f * mu * (tF[3 * i + j] - tD[3 * i + j]) + q[j] + jc * cof[3 * i + j];
    }
}

// tau, and Fb += dL/dF for tb = dL/dtau.
__device__ __forceinline__ void ad_stress_vjp(const float H[9], float mu, float lam, const float tb[9], float tau[9],
                                              float Fb[9]) {
    const Sym3 E = left_cauchy_green_minus_I(H);
    const float jm1 = det_minus_one(H), r2 = frob2(E);
    if (wave_needs_eig(r2, jm1)) {
        Polar P;
        ad_polar(H, P);
        ad_tau(H, P, mu, lam, tau);
        ad_tau_vjp(H, P, mu, lam, tb, Fb);
    } else {
        ad_small_stress(E, r2, jm1, mu, lam, tau);
        ad_small_stress_vjp(H, E, r2, jm1, mu, lam, tb, Fb);
    }
}

__device__ __forceinline__ void load_planes(const float *base, long long stride, int p, int first, int count, float *out) {
    for (int i = 0; i < count; ++i) out[i] = base[(first + i) * stride + p];
}

// ------------------------------------------------------------ workgroup node tiles
// The two scattering kernels accumulate into a 64-bit fixed-point LDS tile over the
// node boxes of their workgroup's 128 particles (both grids), then add every nonzero
// node to the grid with one float atomic per channel.  Particles keep their creation
// order, cell by cell, so consecutive particles sit in neighbouring cells and the box is
// small (a row of about 18 x 3 x 3 nodes for the box workload).  Where a workgroup's
// particles run over the end of a layer or a row of the body, one box over all of them
// can be too large; they are then split in two where consecutive particles first jump by
// more than three cells in y, or else in x (a body of 27 x 24 cells: one workgroup in
// twenty ran over the end of a layer; its direct additions made P2G of 119,223 particles
// 68 us instead of 29.5).  A workgroup whose boxes do not fit either way adds its contributions to the
// grid directly.  Integer sums are exact; the unit is 2^-39 of the largest contribution
// bound of the workgroup, so a node's sum of at most 128 contributions stays below 2^47.
constexpr int kAdTileWords = 5120;   // 40 KiB
constexpr int kAdParticles = 128;    // particles of a 256-thread workgroup
constexpr int kAdTileInts = 16;      // LDS ints of the tile's set-up

struct AdTile {
    unsigned long long *w;        // [channel][grid][T]
    int lo[2][3], L[2][3], off1, T;   // the boxes; the second one's first node, nodes of both
    bool on;
    double S;
};

// round(v S) as a two's-complement 64-bit integer (|v S| < 2^51): in [2^52, 2^53) the
// FP64 numbers are the integers, so magic + v S carries it in its low bits.
__device__ __forceinline__ unsigned long long ad_fixed(float v, double S) {
    constexpr double kMagic = 6755399441055744.0;   // 1.5 * 2^52
    return (unsigned long long)(__double_as_longlong(fma((double)v, S, kMagic)) - 0x4338000000000000LL);
}

// Minimum of v over the wave's lanes, added to *at by its last lane (lane exchanges within
// the vector registers: rows of 16 by shifts, then row to row).
__device__ __forceinline__ void ad_wave_min(int v, int *at) {
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x111, 0xF, 0xF, false));   // row_shr 1, 2, 4, 8
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x112, 0xF, 0xF, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x114, 0xF, 0xF, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x118, 0xF, 0xF, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x142, 0xA, 0xF, false));   // row_bcast 15, 31
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x143, 0xC, 0xF, false));
    if ((threadIdx.x & 63) == 63) atomicMin(at, v);
}

// Node box of the lanes for which `in` holds, into box k of the tile (lo and, negated,
// hi in sh[6 k ..]); every thread calls it between barriers.
__device__ __forceinline__ void ad_box(bool in, const AdStencil &st, int *sh) {
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        ad_wave_min(in ? st.base[ax] : INT_MAX, &sh[ax]);
        ad_wave_min(in ? -st.base[ax] - 1 : INT_MAX, &sh[3 + ax]);
    }
}

// Box k from sh; returns its node count (0 when it is empty).
__device__ __forceinline__ long long ad_box_read(const int *sh, int k, AdTile &t) {
    long long T = 1;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        t.lo[k][ax] = sh[ax];
        t.L[k][ax] = sh[ax] == INT_MAX ? 0 : -sh[3 + ax] - sh[ax] + 1;
        T *= t.L[k][ax];
    }
    return T;
}

// Called by every thread of the workgroup: node boxes of the valid particles' stencils on
// both grids, scale from the largest bound `bnd`, tile of `nch` channels cleared when it
// fits; sel: the thread's box.  sh: kAdTileInts ints of LDS.
__device__ void ad_tile_begin(bool valid, const AdStencil &st, float bnd, int nch, unsigned long long *words, int *sh,
                              AdTile &t, int &sel) {
    const int tid = threadIdx.x;
    sel = 0;
    if (tid < kAdTileInts) sh[tid] = INT_MAX;
    __syncthreads();
    ad_box(valid, st, sh);
    // the largest bound as the smallest negated bit pattern (bounds are not negative)
    ad_wave_min(valid ? -__float_as_int(bnd) : 0, &sh[12]);
    __syncthreads();
    t.w = words;
    long long T0 = ad_box_read(sh, 0, t), T1 = 0;
    const bool any = sh[0] != INT_MAX;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        t.lo[1][ax] = 0;
        t.L[1][ax] = 0;
    }
    int *at = reinterpret_cast<int *>(words);   // the tile's words are not in use yet
    for (int ax = 1; ax >= 0 && any && 2 * (T0 + T1) * nch > kAdTileWords; --ax) {
        __syncthreads();   // the boxes have been read
        at[tid] = valid ? st.base[ax] : INT_MIN;
        if (tid < 12) sh[tid] = INT_MAX;
        if (tid == 13) sh[13] = INT_MAX;
        __syncthreads();
        if (valid && tid >= 2 && at[tid - 2] != INT_MIN && abs(st.base[ax] - at[tid - 2]) > 3) atomicMin(&sh[13], tid & ~1);
        __syncthreads();
        sel = tid >= sh[13] ? 1 : 0;
        ad_box(valid && !sel, st, sh);
        ad_box(valid && sel, st, sh + 6);
        __syncthreads();
        T0 = ad_box_read(sh, 0, t);
        T1 = ad_box_read(sh + 6, 1, t);
    }
    t.on = any && 2 * (T0 + T1) * nch <= kAdTileWords;
    t.off1 = t.on ? (int)T0 : 0;
    t.T = t.on ? (int)(T0 + T1) : 0;
    const float m = __int_as_float(-sh[12]);
    t.S = m > 0.0f ? ldexp(1.0, 39 - ilogbf(m)) : 1.0;
    if (t.on)
        for (int q = tid; q < 2 * t.T * nch; q += blockDim.x) words[q] = 0ull;
    __syncthreads();
}

// Tile position of the lane's base node and the steps to the next node in y and z.
__device__ __forceinline__ int ad_tile_base(const AdTile &t, const AdStencil &st, int sel, int &sy, int &sz) {
    const int l0 = sel ? t.lo[1][0] : t.lo[0][0], l1 = sel ? t.lo[1][1] : t.lo[0][1], l2 = sel ? t.lo[1][2] : t.lo[0][2];
    sy = sel ? t.L[1][0] : t.L[0][0];
    sz = sy * (sel ? t.L[1][1] : t.L[0][1]);
    return pair_grid() * t.T + (sel ? t.off1 : 0) + (st.base[2] - l2) * sz + (st.base[1] - l1) * sy + (st.base[0] - l0);
}

// v of lane `from` of the four consecutive lanes.
template <int kFrom>
__device__ __forceinline__ int quad_lane(int v) {
    return __builtin_amdgcn_update_dpp(0, v, 0x55 * kFrom, 0xF, 0xF, true);   // quad_perm from, from, from, from
}

// Adds lane kFrom's c[0 .. nch) at its node id (none when negative), one channel per lane of
// the four.
template <int kFrom>
__device__ __forceinline__ void ad_add_quad(float4 *x, long long id, const float (&c)[4], int nch) {
    const int lo = quad_lane<kFrom>((int)id), hi = quad_lane<kFrom>((int)(id >> 32)), ch = (int)threadIdx.x & 3;
    float v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = __int_as_float(quad_lane<kFrom>(__float_as_int(c[k])));
    const float mine = ch == 0 ? v[0] : ch == 1 ? v[1] : ch == 2 ? v[2] : v[3];
    const long long at = (long long)((unsigned long long)(unsigned int)hi << 32 | (unsigned int)lo);
    if (hi >= 0 && ch < nch) atomicAdd(reinterpret_cast<float *>(x + at) + ch, mine);
}

// Every lane's contribution to a node straight to the node array x, for workgroups whose tile
// is off (every lane calls it; id negative: none).  Four consecutive lanes take the four
// channels of one of their nodes at a time, as in the flush: with a lane's four channels one
// after the other, a wave's every atomic met 64 cache lines instead of 16 (65,536 particles
// in random order: P2G 399 us against 110, G2P adjoint 272 against 103).
__device__ __forceinline__ void ad_add(float4 *x, long long id, const float (&c)[4], int nch) {
    ad_add_quad<0>(x, id, c, nch);
    ad_add_quad<1>(x, id, c, nch);
    ad_add_quad<2>(x, id, c, nch);
    ad_add_quad<3>(x, id, c, nch);
}

// Called by every thread after its adds: every nonzero value of the tile to the node
// array x.  Four consecutive lanes take a node's channels, so that a wave's atomics go to
// consecutive addresses.
template <bool kSparse>
__device__ void ad_tile_flush(const AdArgs &a, const AdTile &t, float4 *x, int nch) {
    __syncthreads();
    if (!t.on) return;
    const double inv = 1.0 / t.S;
    const int ch = threadIdx.x & 3;
    for (int q = threadIdx.x >> 2; q < 2 * t.T; q += blockDim.x >> 2) {
        const int g = q >= t.T ? 1 : 0, rt = q - g * t.T, k = rt >= t.off1 ? 1 : 0;
        const long long v = ch < nch ? (long long)t.w[(ch * 2 + g) * t.T + rt] : 0ll;
        if (v == 0) continue;
        const int r = rt - (k ? t.off1 : 0), L0 = k ? t.L[1][0] : t.L[0][0], L1 = k ? t.L[1][1] : t.L[0][1];
        // r / L0 and so on through FP32: exact for these sizes (r < 2^13)
        const int row = (int)(((float)r + 0.5f) / (float)L0), iz = (int)(((float)row + 0.5f) / (float)L1);
        const long long id = ad_index<kSparse>(a, g, (k ? t.lo[1][0] : t.lo[0][0]) + r - row * L0,
                                               (k ? t.lo[1][1] : t.lo[0][1]) + row - iz * L1,
                                               (k ? t.lo[1][2] : t.lo[0][2]) + iz);
        atomicAdd(reinterpret_cast<float *>(x + id) + ch, (float)((double)v * inv));
    }
}

// ------------------------------------------------------------ kernels
// Clears, for later calls, the X that the call before used (and VB when it holds a
// reverse call's sums): the workgroups of the P2G launch past a.pgrid.
template <bool kSparse>
__device__ void ad_clear(const AdArgs &a, unsigned int use) {
    float4 *x = ad_x(a, use ^ 1u), *vb = ad_vb(a);
    const bool both = a.ctl[A_VB] != 0u;
    const long long t0 = (long long)((int)blockIdx.x - a.pgrid) * 256 + threadIdx.x;
    const long long step = (long long)((int)gridDim.x - a.pgrid) * 256;
    const float4 zero = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        const long long n = kSparse ? 64ll * min(a.ctl[A_PREV + g], (unsigned int)a.cap) : a.nodes;
        for (long long i = t0; i < n; i += step) {
            x[g * a.nodes + i] = zero;
            if (both) vb[g * a.nodes + i] = zero;
        }
    }
}

// P2G through the workgroup's node tile (direct float atomics when it does not fit).
template <bool kSparse>
__global__ void __launch_bounds__(256) k_ad_p2g(AdArgs a, const float *state, const float *logE) {
    __shared__ unsigned long long tw[kAdTileWords];
    __shared__ int sh[kAdTileInts];
    const unsigned int use = a.ctl[A_CUR] & 1u;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.ctl[A_USE] = use;
    if ((int)blockIdx.x >= a.pgrid) {   // the whole workgroup
        ad_clear<kSparse>(a, use);
        return;
    }
    float4 *x4 = ad_x(a, use);
    const int p = ad_block(a) * kAdParticles + (threadIdx.x >> 1);
    float x[3], v[3], Q[9];
    AdStencil st;
    bool valid = false;
    if (p < a.n) {
        float B[9], H[9], xr[3];
        load_planes(state, a.stride, p, 0, 3, x);
        load_planes(state, a.stride, p, 3, 3, v);
        load_planes(state, a.stride, p, 6, 9, B);
        load_planes(state, a.stride, p, 15, 9, H);
        load_planes(state, a.stride, p, kPlaneR, 3, xr);
        const float lE = logE[p];
        valid = ad_stencil(a, x, xr, st);
        if (!valid) {
            ad_status(a, ST_DOMAIN);
        } else {
            const float E = expf(lE);
            float tau[9];
            ad_stress(H, a.nu_mu * E, a.nu_lambda * E, tau);
            float A[9];
#pragma unroll
            for (int i = 0; i < 9; ++i) A[i] = a.mass * B[i] - a.dt * a.vol0 * tau[i];
            mat_mul(A, st.Dinv, Q);
        }
    }
    // |w m| <= m and |w (m v + Q d)| <= |m v| + dx sum |Q| (w <= 1, |d_b| <= dx)
    float bnd = 0.0f;
    if (valid) {
        bnd = a.mass;
#pragma unroll
        for (int ax = 0; ax < 3; ++ax)
            bnd = fmaxf(bnd, fabsf(a.mass * v[ax]) +
                                 a.geo.dx * (fabsf(Q[3 * ax]) + fabsf(Q[3 * ax + 1]) + fabsf(Q[3 * ax + 2])));
    }
    AdTile t;
    int sel;
    ad_tile_begin(valid, st, bnd, 4, tw, sh, t, sel);
    const auto terms = [&](int o, float (&c)[4]) {
        float w, d[3], gw[3];
        ad_weights(a, st, o, w, d, gw);
        c[0] = w * a.mass;
#pragma unroll
        for (int ax = 0; ax < 3; ++ax)
            c[1 + ax] = w * (a.mass * v[ax] + Q[3 * ax] * d[0] + Q[3 * ax + 1] * d[1] + Q[3 * ax + 2] * d[2]);
    };
    if (!t.on) {   // the whole workgroup
        for (int i = 0; i < 8; ++i) {
            const int o = ad_turn(i);
            float c[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            long long id = -1;
            if (valid) {
                terms(o, c);
                id = ad_index<kSparse>(a, pair_grid(), st.base[0] + (o & 1), st.base[1] + ((o >> 1) & 1), st.base[2] + (o >> 2));
            }
            ad_add(x4, id, c, 4);
        }
    } else if (valid) {
        int sy, sz;
        const int r0 = ad_tile_base(t, st, sel, sy, sz);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int o = ad_turn(i), ox = o & 1, oy = (o >> 1) & 1, oz = o >> 2;
            float c[4];
            terms(o, c);
            unsigned long long *tp = t.w + r0 + ox + oy * sy + oz * sz;
#pragma unroll
            for (int ch = 0; ch < 4; ++ch) atomicAdd(tp + ch * 2 * t.T, ad_fixed(c[ch], t.S));
        }
    }
    ad_tile_flush<kSparse>(a, t, x4, 4);
}

// Marks the blocks of the nodes a valid particle's stencil reaches on both grids
// (nodes base and base + 1 per axis, base = floor(X - k/4) as in ad_stencil).
// Also keeps the previous call's slot counts (for the clearing) and zeroes the counters
// that k_ad_alloc then counts up.
__global__ void __launch_bounds__(256) k_ad_mark(AdArgs a, const float *state) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < 2) {
        a.ctl[A_PREV + p] = a.ctl[A_CNT + p];
        a.ctl[A_CNT + p] = 0u;
    }
    if (p >= a.n) return;
    float x[3], xr[3], X[3];
    load_planes(state, a.stride, p, 0, 3, x);
    load_planes(state, a.stride, p, kPlaneR, 3, xr);
    if (!ad_position(a, x, xr, X)) return;
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        const float k = g == 0 ? -0.25f : 0.25f;
        int lo[3], hi[3];
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            const float Xk = X[ax] - k;
            const int b = (int)floorf(Xk);
            lo[ax] = b >> 2;
            hi[ax] = (b + 1) >> 2;
        }
        for (int bz = lo[2]; bz <= hi[2]; ++bz)
            for (int by = lo[1]; by <= hi[1]; ++by)
                for (int bx = lo[0]; bx <= hi[0]; ++bx)
                    a.flag[g * a.nbv + ((long long)bz * a.nby + by) * a.nbx + bx] = 1;
    }
}

// One thread per block of grid blockIdx.y: a marked block takes the grid's next pool
// slot (one counter update per wave); its flag is cleared.
// Every block's page entry is rewritten (-1 for an untouched one).
__global__ void __launch_bounds__(256) k_ad_alloc(AdArgs a) {
    const int g = blockIdx.y;
    const long long b = blockIdx.x * 256LL + threadIdx.x;
    const bool in = b < a.nbv;
    const bool f = in && a.flag[g * a.nbv + b] != 0;
    const unsigned long long m = __ballot(f);
    if (m == 0ull) {
        if (in) a.page[g * a.nbv + b] = -1;
        return;
    }
    const int lane = threadIdx.x & 63, leader = __builtin_ctzll(m);
    unsigned int base = 0u;
    if (lane == leader) base = atomicAdd(&a.ctl[A_CNT + g], (unsigned int)__popcll(m));
    base = __shfl(base, leader);
    if (!in) return;
    int slot = -1;
    if (f) {
        const unsigned int s = base + (unsigned int)__popcll(m & ((1ull << lane) - 1ull));
        if (s < (unsigned int)a.cap) {
            slot = (int)s;
        } else {
            slot = a.cap;
            ad_status(a, ST_CAPACITY);
        }
        a.flag[g * a.nbv + b] = 0;
    }
    a.page[g * a.nbv + b] = slot;
}

template <bool kSparse>
__global__ void __launch_bounds__(256) k_ad_g2p(AdArgs a, const float *state, float *out) {
    const int p = ad_block(a) * kAdParticles + (threadIdx.x >> 1), g = pair_grid();
    const unsigned int use = a.ctl[A_USE];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.ctl[A_CUR] = use ^ 1u;
        a.ctl[A_VB] = 0u;
    }
    if (p >= a.n) return;
    const float4 *x4 = ad_x(a, use);
    float x[3], xr[3], H[9];
    load_planes(state, a.stride, p, 0, 3, x);
    load_planes(state, a.stride, p, kPlaneR, 3, xr);
    load_planes(state, a.stride, p, 15, 9, H);
    AdStencil st;
    if (!ad_stencil(a, x, xr, st)) {
        ad_status(a, ST_DOMAIN);
        for (int i = g; i < MPM_STATE_PLANES; i += 2) out[i * a.stride + p] = state[i * a.stride + p];
        return;
    }
    float vp[3] = {0.0f, 0.0f, 0.0f}, Bn[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) Bn[i] = 0.0f;
    {
        const bool all_free = ad_all_free(a, st);
        long long id[8];
        float4 q[8];
        ad_ids<kSparse>(a, st, id);
        ad_gather(x4, id, q);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int o = ad_turn(i);
            float w, d[3], gw[3], vi[3];
            ad_weights(a, st, o, w, d, gw);
            ad_node_velocity(a, st, all_free, o, q[i], vi);
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                const float wv = 0.5f * w * vi[ax];
                vp[ax] += wv;
#pragma unroll
                for (int b = 0; b < 3; ++b) Bn[3 * ax + b] += wv * d[b];
            }
        }
    }
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) vp[ax] = pair_sum(vp[ax]);
#pragma unroll
    for (int i = 0; i < 9; ++i) Bn[i] = pair_sum(Bn[i]);
    float C[9];
    mat_mul(Bn, st.Dinv, C);
    // the new state's planes; the pair's lanes store half of them each
    float q[28];
    // F' = (I + dt C) F  ->  H' = H + dt C (I + H)
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            q[15 + 3 * i + j] = H[3 * i + j] + a.dt * (C[3 * i + j] + C[3 * i] * H[j] + C[3 * i + 1] * H[3 + j] + C[3 * i + 2] * H[6 + j]);
    float probe = 0.0f;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        advance_position(x[ax], xr[ax], a.dt * vp[ax], q[ax], q[kPlaneR + ax]);
        q[3 + ax] = vp[ax];
        probe += vp[ax] * 0.0f;
    }
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        q[6 + i] = Bn[i];
        probe += Bn[i] * 0.0f + q[15 + i] * 0.0f;
    }
    q[27] = 0.0f;
    float *op = out + (long long)(g ? 14 : 0) * a.stride + p;
#pragma unroll
    for (int i = 0; i < 14; ++i) {
        const float v = g ? q[14 + i] : q[i];
        if (i < 13 || g == 0) *op = v;
        op += a.stride;
    }
    if (!(probe == 0.0f)) ad_status(a, ST_NONFINITE);
}

// G2P reversed: scatters dL/dv~ to the grid, writes the G2P part of dL/dx and dL/dF.
template <bool kSparse>
__global__ void __launch_bounds__(256) k_ad_g2p_vjp(AdArgs a, const float *state, const float *cot_out,
                                                    float *cot_in) {
    __shared__ unsigned long long tw[kAdTileWords];
    __shared__ int sh[kAdTileInts];
    const int p = ad_block(a) * kAdParticles + (threadIdx.x >> 1), lane_g = pair_grid();
    const unsigned int use = a.ctl[A_USE];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.ctl[A_CUR] = use ^ 1u;
        a.ctl[A_VB] = 1u;
    }
    const float4 *x4 = ad_x(a, use);
    float4 *vb4 = ad_vb(a);
    float x[3], xr[3], H[9];
    float xbo[3], vbo[3], Bbo[9], Fbo[9];
    AdStencil st;
    bool valid = false;
    if (p < a.n) {
        load_planes(state, a.stride, p, 0, 3, x);
        load_planes(state, a.stride, p, kPlaneR, 3, xr);
        load_planes(state, a.stride, p, 15, 9, H);
        load_planes(cot_out, a.stride, p, 0, 3, xbo);
        load_planes(cot_out, a.stride, p, 3, 3, vbo);
        load_planes(cot_out, a.stride, p, 6, 9, Bbo);
        load_planes(cot_out, a.stride, p, 15, 9, Fbo);
        valid = ad_stencil(a, x, xr, st);
        if (!valid) {
            // the forward step left this particle unchanged; the position cotangent
            // is that of the x planes, written to the r planes as well
            ad_status(a, ST_DOMAIN);
            for (int i = 0; i < kPlaneR; ++i) cot_in[i * a.stride + p] = cot_out[i * a.stride + p];
            for (int i = 0; i < 3; ++i) cot_in[(kPlaneR + i) * a.stride + p] = xbo[i];
        }
    }
    // Every thread reaches the tile's set-up and flush (they hold workgroup barriers)
    // at the same two points, whatever its particle; invalid lanes add nothing.
    float xb[3], vbt[3], Bbt[9], Cb[9];
    float bnd = 0.0f;
    if (valid) {
        // x' = x + dt v'  ->  xb = xb',  v'b = vb' + dt xb'
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            xb[ax] = lane_g ? 0.0f : xbo[ax];   // a lane's share; summed over the pair below
            vbt[ax] = vbo[ax] + a.dt * xbo[ax];
        }
        // F' = (I + dt C) F  ->  Cb = dt Fb' F^T;  C = B' D^-1  ->  B'b += Cb D^-T
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                float cb = 0.0f;
#pragma unroll
                for (int k = 0; k < 3; ++k) cb += Fbo[3 * i + k] * (H[3 * j + k] + (j == k ? 1.0f : 0.0f));
                Cb[3 * i + j] = a.dt * cb;
            }
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j)
                Bbt[3 * i + j] = Bbo[3 * i + j] + Cb[3 * i] * st.Dinv[3 * j] + Cb[3 * i + 1] * st.Dinv[3 * j + 1] +
                                 Cb[3 * i + 2] * st.Dinv[3 * j + 2];
        // |1/2 w (v'b + B'b d)| <= 1/2 (|v'b| + dx sum |B'b|)
#pragma unroll
        for (int ax = 0; ax < 3; ++ax)
            bnd = fmaxf(bnd, 0.5f * (fabsf(vbt[ax]) + a.geo.dx * (fabsf(Bbt[3 * ax]) + fabsf(Bbt[3 * ax + 1]) +
                                                                  fabsf(Bbt[3 * ax + 2]))));
    }
    AdTile t;
    int sel;
    ad_tile_begin(valid, st, bnd, 3, tw, sh, t, sel);
    if (!t.on) {   // the whole workgroup
        for (int i = 0; i < 8; ++i) {
            const int o = ad_turn(i);
            float c[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            long long at = -1;
            if (valid) {
                float w, d[3], gw[3];
                ad_weights(a, st, o, w, d, gw);
#pragma unroll
                for (int ax = 0; ax < 3; ++ax)
                    c[ax] = 0.5f * w * (vbt[ax] + Bbt[3 * ax] * d[0] + Bbt[3 * ax + 1] * d[1] + Bbt[3 * ax + 2] * d[2]);
                at = ad_index<kSparse>(a, lane_g, st.base[0] + (o & 1), st.base[1] + ((o >> 1) & 1), st.base[2] + (o >> 2));
            }
            ad_add(vb4, at, c, 3);
        }
    }
    if (valid) {
        // one pass over the nodes: the forward B' (for C and (D^-1)b), and
        // v' = 1/2 sum w v~,  B' = 1/2 sum w v~ d^T:
        //   v~b_i += 1/2 w (v'b + B'b d),  wb = 1/2 v~ . (v'b + B'b d),  db = 1/2 w B'b^T v~,
        //   and d = x_i - x_p moves against x_p
        float Bn[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) Bn[i] = 0.0f;
        const bool all_free = ad_all_free(a, st);
        long long id[8];
        float4 q[8];
        ad_ids<kSparse>(a, st, id);
        ad_gather(x4, id, q);
        int sy = 0, sz = 0;
        const int r0 = t.on ? ad_tile_base(t, st, sel, sy, sz) : 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int o = ad_turn(i), ox = o & 1, oy = (o >> 1) & 1, oz = o >> 2;
            float w, d[3], gw[3], vi[3], gv[3];
            ad_weights(a, st, o, w, d, gw);
            ad_node_velocity(a, st, all_free, o, q[i], vi);
            float wb = 0.0f;
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                gv[ax] = vbt[ax] + Bbt[3 * ax] * d[0] + Bbt[3 * ax + 1] * d[1] + Bbt[3 * ax + 2] * d[2];
                wb += 0.5f * vi[ax] * gv[ax];
#pragma unroll
                for (int b = 0; b < 3; ++b) Bn[3 * ax + b] += 0.5f * w * vi[ax] * d[b];
            }
            if (t.on) {
                unsigned long long *tp = t.w + r0 + ox + oy * sy + oz * sz;
#pragma unroll
                for (int ax = 0; ax < 3; ++ax) atomicAdd(tp + ax * 2 * t.T, ad_fixed(0.5f * w * gv[ax], t.S));
            }
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const float db = 0.5f * w * (Bbt[b] * vi[0] + Bbt[3 + b] * vi[1] + Bbt[6 + b] * vi[2]);
                xb[b] += wb * gw[b] - db;
            }
        }
#pragma unroll
        for (int i = 0; i < 9; ++i) Bn[i] = pair_sum(Bn[i]);
        // Fb = (I + dt C)^T Fb',  C = B' D^-1;  (D^-1)b = B'^T Cb
        float C[9], Fb[9], Dib[9];
        mat_mul(Bn, st.Dinv, C);
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                float fb = Fbo[3 * i + j];
#pragma unroll
                for (int k = 0; k < 3; ++k) fb += a.dt * C[3 * k + i] * Fbo[3 * k + j];
                Fb[3 * i + j] = fb;
            }
        mat_tmul(Bn, Cb, Dib);
        float Db[9];
        ad_inverse_vjp(st.Dinv, Dib, Db);
        ad_moment_vjp(a, st, Db, xb);
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            xb[ax] = pair_sum(xb[ax]);
            if (lane_g == 0) cot_in[ax * a.stride + p] = xb[ax];
        }
        if (lane_g) {
#pragma unroll
            for (int i = 0; i < 9; ++i) cot_in[(15 + i) * a.stride + p] = Fb[i];
        }
    }
    ad_tile_flush<kSparse>(a, t, vb4, 3);
}

// P2G and grid update reversed (a gather): on live nodes pb = v~b / m and
// mb = -(v~b . p) / m^2; completes dL/dx and dL/dF, writes dL/dv, dL/dB, adds dL/dlogE.
template <bool kSparse>
__global__ void __launch_bounds__(256) k_ad_p2g_vjp(AdArgs a, const float *state, const float *logE, float *cot_in,
                                                    float *logE_cot) {
    const int p = ad_block(a) * kAdParticles + (threadIdx.x >> 1), g = pair_grid();
    if (p >= a.n) return;
    float x[3], xr[3], v[3], B[9], H[9];
    load_planes(state, a.stride, p, 0, 3, x);
    load_planes(state, a.stride, p, kPlaneR, 3, xr);
    load_planes(state, a.stride, p, 3, 3, v);
    load_planes(state, a.stride, p, 6, 9, B);
    load_planes(state, a.stride, p, 15, 9, H);
    AdStencil st;
    if (!ad_stencil(a, x, xr, st)) return;   // cotangent already passed through by the G2P adjoint
    const float E = expf(logE[p]);
    const float mu = a.nu_mu * E, lam = a.nu_lambda * E;
    const float4 *x4 = ad_x(a, a.ctl[A_USE]), *vb4 = ad_vb(a);
    float A[9], Q[9];
    ad_stress(H, mu, lam, A);
#pragma unroll
    for (int i = 0; i < 9; ++i) A[i] = a.mass * B[i] - a.dt * a.vol0 * A[i];
    mat_mul(A, st.Dinv, Q);
    float xb[3] = {0.0f, 0.0f, 0.0f}, vb[3] = {0.0f, 0.0f, 0.0f}, Qb[9];   // the lane's share
#pragma unroll
    for (int i = 0; i < 9; ++i) Qb[i] = 0.0f;
    const bool all_free = ad_all_free(a, st);
    // m_i += w m,  p_i += w (m v + Q d):
    //   wb = m mb_i + pb_i . (m v + Q d),  vb += w m pb_i,  Qb += w pb_i d^T,  db = w Q^T pb_i
    long long id[8];
    ad_ids<kSparse>(a, st, id);
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        float4 q[4], r[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) q[i] = x4[id[4 * half + i]];
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = vb4[id[4 * half + i]];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int o = ad_turn(4 * half + i);
            float w, d[3], gw[3], vi[3];
            ad_weights(a, st, o, w, d, gw);
            const float im = ad_node_velocity(a, st, all_free, o, q[i], vi);
            const float pb[3] = {r[i].x * im, r[i].y * im, r[i].z * im};
            const float mb = -(r[i].x * q[i].y + r[i].y * q[i].z + r[i].z * q[i].w) * im * im;
            float wb = a.mass * mb;
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                const float pi = a.mass * v[ax] + Q[3 * ax] * d[0] + Q[3 * ax + 1] * d[1] + Q[3 * ax + 2] * d[2];
                wb += pb[ax] * pi;
                vb[ax] += w * a.mass * pb[ax];
#pragma unroll
                for (int b = 0; b < 3; ++b) Qb[3 * ax + b] += w * pb[ax] * d[b];
            }
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const float db = w * (Q[b] * pb[0] + Q[3 + b] * pb[1] + Q[6 + b] * pb[2]);
                xb[b] += wb * gw[b] - db;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 9; ++i) Qb[i] = pair_sum(Qb[i]);
    // Q = A D^-1  ->  Ab = Qb D^-T,  (D^-1)b = A^T Qb
    float Ab[9], Dib[9], Db[9];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            Ab[3 * i + j] = Qb[3 * i] * st.Dinv[3 * j] + Qb[3 * i + 1] * st.Dinv[3 * j + 1] + Qb[3 * i + 2] * st.Dinv[3 * j + 2];
    mat_tmul(A, Qb, Dib);
    ad_inverse_vjp(st.Dinv, Dib, Db);
    ad_moment_vjp(a, st, Db, xb);
    // stored as soon as they are known; the pair's lanes store half of the planes each
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const float xs = cot_in[ax * a.stride + p] + pair_sum(xb[ax]), vs = pair_sum(vb[ax]);
        // the position is x + r: both take its cotangent
        cot_in[(g ? kPlaneR + ax : ax) * a.stride + p] = xs;
        if (g == 0) cot_in[(3 + ax) * a.stride + p] = vs;
    }
#pragma unroll
    for (int i = 0; i < 9; ++i)
        if ((i < 5) == (g == 0)) cot_in[(6 + i) * a.stride + p] = a.mass * Ab[i];
    // A = m B - dt V0 tau  ->  Bb = m Ab,  taub = -dt V0 Ab.  H is read again rather than
    // held through the gather.
    float tb[9], Fb[9], tau[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) tb[i] = -a.dt * a.vol0 * Ab[i];
    load_planes(state, a.stride, p, 15, 9, H);
    load_planes(cot_in, a.stride, p, 15, 9, Fb);
    ad_stress_vjp(H, mu, lam, tb, tau, Fb);
    if (g) {
#pragma unroll
        for (int i = 0; i < 9; ++i) cot_in[(15 + i) * a.stride + p] = Fb[i];
    } else {
        float lb = 0.0f;
#pragma unroll
        for (int i = 0; i < 9; ++i) lb += tb[i] * tau[i];   // tau is proportional to E = exp(logE)
        logE_cot[p] += lb;
    }
}

AdArgs make_args(const mpm_ad_ctx *c, int64_t n, int64_t stride, double dt) {
    AdArgs a;
    a.geo = c->geo;
    for (int i = 0; i < 3; ++i) a.g[i] = c->gravity[i];
    a.mass = c->rho * c->vol0;
    a.vol0 = c->vol0;
    a.nu_mu = (float)(1.0 / (2.0 * (1.0 + c->nu)));
    a.nu_lambda = (float)(c->nu / ((1.0 + c->nu) * (1.0 - 2.0 * c->nu)));
    a.nbx = c->nb[0];
    a.nby = c->nb[1];
    a.cap = c->cap;
    a.nbv = c->nbv;
    a.nodes = c->nodes;
    a.nx = c->geo.n[0] + 1;
    a.ny = c->geo.n[1] + 1;
    a.grid = c->grid;
    a.page = c->page;
    a.direct = c->direct ? 1 : 0;
    a.flag = c->flag;
    a.ctl = c->ctl;
    a.status = c->status;
    a.n = (int)n;
    a.pgrid = (int)((n + 8 * kAdParticles - 1) / (8 * kAdParticles)) * 8;
    a.stride = stride;
    a.dt = (float)dt;
    return a;
}

// Workgroups that clear a call's leftover arrays: eight nodes per thread, at most 1024.
int clear_blocks(const AdArgs &a) {
    const long long nodes = a.direct ? 2 * a.nodes : 2ll * a.cap * 64;
    return (int)std::min<long long>(1024, (nodes + 2047) / 2048);
}

// Blocks marked and given slots (unless direct), then P2G.  n > 0.
void enqueue_p2g(const AdArgs &a, const float *state, const float *logE, hipStream_t s) {
    const dim3 wg(256), grid(a.pgrid + clear_blocks(a));
    if (a.direct) {
        hipLaunchKernelGGL(k_ad_p2g<false>, grid, wg, 0, s, a, state, logE);
    } else {
        hipLaunchKernelGGL(k_ad_mark, dim3((a.n + 255) / 256), wg, 0, s, a, state);
        hipLaunchKernelGGL(k_ad_alloc, dim3((unsigned int)((a.nbv + 255) / 256), 2), wg, 0, s, a);
        hipLaunchKernelGGL(k_ad_p2g<true>, grid, wg, 0, s, a, state, logE);
    }
}

void free_buffers(mpm_ad_ctx *c) {
    void *bufs[] = {c->grid, c->page, c->flag, c->ctl, c->status};
    for (void *b : bufs)
        if (b) (void)hipFree(b);
}

mpm_status check_call(const mpm_ad_ctx *c, int64_t n, int64_t stride, const float *state, double dt) {
    if (!c || n < 0 || n > c->max_particles || stride < n) return MPM_E_INVALID;
    if (n > 0 && !state) return MPM_E_INVALID;
    if (!std::isfinite(dt) || dt < 0) return MPM_E_INVALID;
    return MPM_OK;
}

}  // namespace

extern "C" {

mpm_status mpm_ad_create(const mpm_config *cfg, const mpm_material *mat, mpm_ad_ctx **out) {
    if (!out) return MPM_E_INVALID;
    *out = nullptr;
    if (check_config(cfg, mat, 1) != MPM_OK || mat->model != MPM_FIXED_COROTATED) return MPM_E_INVALID;
    mpm_ad_ctx *c = new (std::nothrow) mpm_ad_ctx();
    if (!c) return MPM_E_OOM;
    if (hipGetDevice(&c->device) != hipSuccess) {
        delete c;
        return MPM_E_HIP;
    }
    geometry_of(*cfg, c->geo);
    for (int i = 0; i < 3; ++i) c->gravity[i] = (float)cfg->gravity[i];
    c->nu = mat->nu;
    c->rho = mat->rho;
    c->vol0 = mat->vol0;
    c->max_particles = cfg->max_particles;
    c->nbv = 1;
    for (int i = 0; i < 3; ++i) {
        c->nb[i] = cfg->n_cells[i] / 4 + 1;
        c->nbv *= c->nb[i];
    }
    c->cap = (int)std::min<long long>(cfg->max_blocks, c->nbv);
    c->direct = c->cap == c->nbv;
    c->nodes = c->direct ? (long long)(cfg->n_cells[0] + 1) * (cfg->n_cells[1] + 1) * (cfg->n_cells[2] + 1)
                         : (long long)(c->cap + 1) * 64;
    const size_t bytes = 3 * 2 * (size_t)c->nodes * sizeof(float4);
    const size_t nbv2 = 2 * (size_t)c->nbv;
    bool ok = hipMalloc(&c->grid, bytes) == hipSuccess && hipMalloc(&c->ctl, kCtlWords * sizeof(unsigned int)) == hipSuccess &&
              hipMalloc(&c->status, sizeof(unsigned int)) == hipSuccess;
    if (!c->direct)   // page tables and marks of the block-sparse pool
        ok = ok && hipMalloc(&c->page, nbv2 * sizeof(int)) == hipSuccess && hipMalloc(&c->flag, nbv2) == hipSuccess && hipMemset(c->flag, 0, nbv2) == hipSuccess;
    // the scatter targets start at zero, and every call clears what the call before left
    // in the arrays that the next one uses; no block is marked between calls
    ok = ok && hipMemset(c->grid, 0, bytes) == hipSuccess &&
         hipMemset(c->ctl, 0, kCtlWords * sizeof(unsigned int)) == hipSuccess &&
         hipMemset(c->status, 0, sizeof(unsigned int)) == hipSuccess;
    if (!ok) {
        free_buffers(c);
        delete c;
        return MPM_E_OOM;
    }
    *out = c;
    return MPM_OK;
}

mpm_status mpm_ad_destroy(mpm_ad_ctx *c) {
    if (!c) return MPM_E_INVALID;
    (void)hipSetDevice(c->device);
    (void)hipDeviceSynchronize();
    free_buffers(c);
    delete c;
    return MPM_OK;
}

mpm_status mpm_ad_forward(mpm_ad_ctx *c, int64_t n, int64_t stride, const float *state_in, const float *logE,
                          float *state_out, double dt, void *stream) {
    const mpm_status v = check_call(c, n, stride, state_in, dt);
    if (v != MPM_OK) return v;
    if (n > 0 && (!logE || !state_out)) return MPM_E_INVALID;
    if (hipSetDevice(c->device) != hipSuccess) return MPM_E_HIP;
    hipStream_t s = (hipStream_t)stream;
    const AdArgs a = make_args(c, n, stride, dt);
    if (n > 0) {
        const dim3 pg(a.pgrid), wg(256);
        enqueue_p2g(a, state_in, logE, s);
        if (a.direct) hipLaunchKernelGGL(k_ad_g2p<false>, pg, wg, 0, s, a, state_in, state_out);
        else hipLaunchKernelGGL(k_ad_g2p<true>, pg, wg, 0, s, a, state_in, state_out);
    }
    return hipGetLastError() == hipSuccess ? MPM_OK : MPM_E_HIP;
}

mpm_status mpm_ad_backward(mpm_ad_ctx *c, int64_t n, int64_t stride, const float *state_in, const float *logE,
                           const float *cot_out, float *cot_in, float *logE_cot, double dt, void *stream) {
    const mpm_status v = check_call(c, n, stride, state_in, dt);
    if (v != MPM_OK) return v;
    if (n > 0 && (!logE || !cot_out || !cot_in || !logE_cot)) return MPM_E_INVALID;
    if (hipSetDevice(c->device) != hipSuccess) return MPM_E_HIP;
    hipStream_t s = (hipStream_t)stream;
    const AdArgs a = make_args(c, n, stride, dt);
    if (n > 0) {
        const dim3 pg(a.pgrid), wg(256);
        enqueue_p2g(a, state_in, logE, s);
        if (a.direct) {
            hipLaunchKernelGGL(k_ad_g2p_vjp<false>, pg, wg, 0, s, a, state_in, cot_out, cot_in);
            hipLaunchKernelGGL(k_ad_p2g_vjp<false>, pg, wg, 0, s, a, state_in, logE, cot_in, logE_cot);
        } else {
            hipLaunchKernelGGL(k_ad_g2p_vjp<true>, pg, wg, 0, s, a, state_in, cot_out, cot_in);
            hipLaunchKernelGGL(k_ad_p2g_vjp<true>, pg, wg, 0, s, a, state_in, logE, cot_in, logE_cot);
        }
    }
    return hipGetLastError() == hipSuccess ? MPM_OK : MPM_E_HIP;
}

mpm_status mpm_ad_sync(mpm_ad_ctx *c, void *stream) {
    if (!c) return MPM_E_INVALID;
    if (hipSetDevice(c->device) != hipSuccess) return MPM_E_HIP;
    if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) return MPM_E_HIP;
    unsigned int bits = 0;
    if (hipMemcpy(&bits, c->status, sizeof bits, hipMemcpyDeviceToHost) != hipSuccess) return MPM_E_HIP;
    const unsigned int zero = 0;
    if (bits != 0 && hipMemcpy(c->status, &zero, sizeof zero, hipMemcpyHostToDevice) != hipSuccess) return MPM_E_HIP;
    return status_from_bits(bits);
}

}  // extern "C"
