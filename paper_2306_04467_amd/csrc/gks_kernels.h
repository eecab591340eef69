// Device kernels of one S2O4 stage of the compact gas-kinetic scheme (gfx950, wave64).
//
// Every kernel is a template on R, the precision of the bulk arithmetic and storage: double for
// the FP64 path, float for the mixed path.  Whatever decides the lake-at-rest balance stays in
// double in both: cell thicknesses (h2 and the interface level eta1 = h1 + B), Gauss-point
// thicknesses, the hydrostatic part 1/2 G h^2 of the normal momentum flux, the interface
// thickness, and every edge sum of the cell update (flux divergence, Green-Gauss derivatives,
// sources).  What is computed in R there vanishes exactly at rest by left/right symmetry.
//
// Data layout:
//   state  by cell, then layer (0 upper, 1 lower): LayerW W[TG][2] {h2 or eta1 in double, the two
//          momenta}, LayerG G[TG][2] {x/y gradients of the three}, TG = T + NG ghosts: what the
//          reconstruction gathers of a stencil cell lies in one or two cache lines
//   rec    GpHead[6 T] and GpTail[6 T]: the reconstruction at each cell's six Gauss points, by local
//          edge, then cell (rec_at), read by the edge kernels as 16-byte words
//   eoh    [6][E] double: per edge, Gauss points averaged: 1/2 G hb^2 (upper, lower), hb (upper,
//          lower), hb the interface thickness of the evolution, then the mean of the two sides'
//          reconstructed thicknesses (upper, lower) for the layer coupling
//   eom    [24][E] R: F0 (6, hydrostatic part removed), Ft (6), interface momenta (4), interface
//          time derivatives (6), global frame, then the mean of the two sides' thickness rates
//          (upper, lower); read by the cell update's gather
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gks_mlp.h"

namespace gks {

struct MeshDev {
    int64_t T, E, NG;
    int32_t S;                      // number of scenarios (independent meshes) in this mesh
    // FP64 tables
    const double *area, *Bbar, *gB, *fl, *gg, *eBgp, *gR, *sdxmin;
    // tables in the bulk precision (double or float copies); M, the least-squares operators, is
    // block-major [ceil(T / RECON_CELLS)][OP_LOADS][RECON_CELLS][4]: entry 9 r + k of a cell's
    // operator (coefficient k, right-hand side r) is entry 4 j + e of that order
    const void *M, *hs, *vtx, *nbc, *en, *egB;
    const float *igeo;              // [6][T] indicator geometry
    const uint8_t *cand;            // [T] plane candidates of the nonlinear reconstruction (bits 0..2)
    const int32_t *cedge, *sten, *eL, *eR, *eslot, *gsrc;
    const int32_t *gfirst, *gof;    // ghosts gof[gfirst[c] .. gfirst[c + 1]) mirror cell c
    const int32_t *cscen, *escen;   // scenario of each cell / edge, nullptr when S == 1
    const int64_t *scell;           // [S + 1] first cell of each scenario
};

struct Phys {
    double G, eps, eps_num, cfl;
    double h_dry;         // wet/dry threshold (0: every layer is wet everywhere)
    int linear;
    int alpha_mode;       // 0: the well-balance weights read here, 1: the paper's printed constants
    const double *chi;    // [S] density ratio
    const double *t_end;  // [S]
    double *scal;         // [2S] per scenario: dt of the current step, time at its end
    // the state's largest wave speeds, left by the second stage's update for the next step: per wave of 32
    // cells of one scenario, and per scenario, as the bits of a non-negative double (whose order is that of
    // the value), the waves that hold a border or the mesh's end (cleared by the step that uses them)
    double *speed;             // [ceil(T / 32)]
    unsigned long long *smax;  // [S]
    unsigned long long *bad;  // smallest cell whose updated state is non-finite or has a layer
                              // thickness <= 0 (all ones: none), kept until the state is reloaded
};

// the force model's weight w is taken as 1 when it is within 1e-12 of 1: the blend would then
// change the acceleration by less than its own FP64 rounding
constexpr double W_ONE = 1.0 - 1e-12;

// Wet/dry layers (Phys::h_dry > 0; the paper's dam breaks over a dry bed, with no treatment given
// there): a side of an interface whose thickness is at or below h_dry is a vacuum, an interface
// whose equilibrium thickness is at or below h_dry passes nothing, and the front band of a layer --
// the cells where the layer, in the cell or in one of its face neighbours, is thinner than
// WD_THIN h_dry or than WD_FRONT times the thickest of the four, and the cells where the lower
// layer is thinner than the bottom's rise across the cell -- is reconstructed at first order and
// evolves at first order in space and time.  Below WD_THIN h_dry a cell's velocity is
// desingularised (Kurganov and Petrova 2007).
constexpr double WD_THIN = 1000.0, WD_FRONT = 0.3;

// a b + c d with one order of rounding in every kernel it is inlined into: what a step leaves for the next
// (ghosts, wave speeds) is also formed from a loaded checkpoint, by other kernels, and has to have the
// same bits there; left to the compiler, either product may be the one that is fused
__host__ __device__ inline double fma2(double a, double b, double c, double d)
{
#pragma clang fp contract(off)
    const double q = c * d;
    return fma(a, b, q);
}

__host__ __device__ inline double wd_velocity(double h, double m, double h_dry)
{
    const double hs = WD_THIN * h_dry;
    if (!(h_dry > 0) || h >= hs) return m / h;
    const double h2 = h * h, d2 = hs * hs;
    return 1.4142135623730950488 * h * m / sqrt(fma2(d2, d2, h2, h2));
}


// relative floor of the smoothness indicators of the nonlinear reconstruction, above the
// rounding of the bulk precision: the weights leave their linear values once a variable varies
// by about 1e-9 of its scale (FP64), 1e-5 in the mixed path, whose reconstruction runs in FP32
template <typename R>
__device__ constexpr R eps_rel()
{
    return sizeof(R) == 8 ? R(1e-18) : R(1e-10);
}

template <typename R>
__device__ inline const R *tab(const void *p)
{
    return static_cast<const R *>(p);
}

// Checked build (GKS_CHECKED): every index read from a mesh table is tested against the size of
// the array it indexes before it is used; a miss sets oob_flag and the access falls back to
// element 0, so the kernel itself stays in bounds.  Other builds take the index as it is.
#ifdef GKS_CHECKED
__device__ unsigned int oob_flag;
__device__ inline int64_t checked_index(int64_t i, int64_t n)
{
    if (i < 0 || i >= n) {
        atomicOr(&oob_flag, 1u);
        return 0;
    }
    return i;
}
#define GKS_IX(i, n) ::gks::checked_index((int64_t)(i), (int64_t)(n))
#else
#define GKS_IX(i, n) (i)
#endif

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own L2.  Cells and edges
// are numbered with spatial locality, so give each XCD one contiguous range of blocks: neighbour
// gathers then hit the same L2 instead of being fetched from HBM by several XCDs.
constexpr int N_XCD = 8;

__device__ inline int64_t xcd_block(unsigned extra = 0)  // blocks of another kind before the kernel's own
{
    const int64_t b = blockIdx.x - extra, nb = gridDim.x - extra;
    const int64_t q = nb / N_XCD, r = nb % N_XCD, x = b % N_XCD, j = b / N_XCD;
    return x * q + (x < r ? x : r) + j;
}

// one layer of a cell: h2 and its momenta, or eta1 = h1 + B and the lower layer's momenta
template <typename R>
struct LayerW {
    double h;
    R m[2];
};

// x / y derivatives of the layer's three variables
template <typename R>
struct LayerG {
    R g[6];
};

// a / b in the bulk precision: in FP32 the product with the hardware reciprocal (one instruction,
// within about an ulp, where the correctly rounded quotient costs about ten; FP32 results are
// held to FP32 tolerances), in FP64 the correctly rounded quotient
__device__ inline float div_(float a, float b) { return a * __builtin_amdgcn_rcpf(b); }
__device__ inline double div_(double a, double b) { return a / b; }

// Gauss-point records of one cell at one of its six Gauss points (slot = 2 * local edge + point),
// written by the reconstruction and read by the edge kernels, in two arrays: the head (thicknesses
// and momenta, all that the force model's edge kernel reads) and the tail (gradients), so that each is
// read as a few 16-byte words.  Both are stored by local edge, then cell, then point (rec_at): the two
// points an edge reads lie side by side, and a block of cells writes whole contiguous spans an
// edge at a time.
//   head.h[0] h2, head.h[1] eta1 = h1 + B (double in both precisions)
//   head.q[0..3]  momenta h2U2, h2V2, h1U1, h1V1
//   tail.g[2 v], tail.g[2 v + 1]  x / y derivative of paper component v (v = 0..5, eta1 for h1)
template <typename R>
struct alignas(16) GpHead {
    double h[2];
    R q[4];
};

template <typename R>
struct alignas(16) GpTail {
    R g[12];
};

template <typename R>
struct GpRecs {
    GpHead<R> *head;
    GpTail<R> *tail;
};

// index of the record of cell c at Gauss point g of its local edge k
__host__ __device__ inline int64_t rec_at(int64_t T, int64_t c, int k, int g) { return 2 * (k * T + c) + g; }


// --------------------------------------------------------------------------------------------
// ghost mirror cells: state of the source cell seen through an orthogonal map

// layer l of ghost cell g from that of its source cell
template <typename R>
__device__ inline void mirror(const MeshDev &m, int64_t g, int l, const LayerW<R> &w, const LayerG<R> &q,
                              LayerW<R> *__restrict__ W, LayerG<R> *__restrict__ G)
{
    const int64_t d = m.T + g, NG = m.NG;
    // R (a b; c e) maps gradient directions, V (va vb; vc ve) momentum vectors: V = R across a
    // wall, V = I across a free boundary (each component extended evenly)
    const double a = m.gR[g], b = m.gR[NG + g], c = m.gR[2 * NG + g], e = m.gR[3 * NG + g];
    const double va = m.gR[4 * NG + g], vb = m.gR[5 * NG + g], vc = m.gR[6 * NG + g], ve = m.gR[7 * NG + g];
    const double mx = w.m[0], my = w.m[1], hx = q.g[0], hy = q.g[1];
    W[2 * d + l] = {w.h, {(R)fma2(va, mx, vb, my), (R)fma2(vc, mx, ve, my)}};
    // momentum gradient G[i][j] = d m_i / d x_j  ->  V G R^T
    const double g00 = q.g[2], g01 = q.g[3], g10 = q.g[4], g11 = q.g[5];
    const double r00 = fma2(va, g00, vb, g10), r01 = fma2(va, g01, vb, g11);
    const double r10 = fma2(vc, g00, ve, g10), r11 = fma2(vc, g01, ve, g11);
    G[2 * d + l] = {{(R)fma2(a, hx, b, hy), (R)fma2(c, hx, e, hy), (R)fma2(r00, a, r01, b), (R)fma2(r00, c, r01, e),
                     (R)fma2(r10, a, r11, b), (R)fma2(r10, c, r11, e)}};
}

// all ghosts of a state that did not come from k_update, which writes them along with its cells
template <typename R>
__global__ void __launch_bounds__(256) k_ghost_fill(MeshDev m, LayerW<R> *__restrict__ W, LayerG<R> *__restrict__ G)
{
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= m.NG) return;
    const int64_t s = GKS_IX(m.gsrc[g], m.T);
#pragma unroll
    for (int l = 0; l < 2; l++) mirror(m, g, l, W[2 * s + l], G[2 * s + l], W, G);
}

// --------------------------------------------------------------------------------------------
// compact reconstruction (Sec. 3.4): one wave per 32 cells, lane l layer l % 2 of cell l / 2

constexpr int RECON_CELLS = 32;
constexpr int OP_LOADS = 39;  // loads of four operator entries per cell (153, padded to 156)

// An operator load brings entries 4 j and 4 j + 1 to a cell's even lane and 4 j + 2 and 4 j + 3 to its
// odd lane; both need all four: each entry is spread over the pair in registers (DPP), so that none is
// fetched or held in flight twice.
template <int ODD>
__device__ inline uint32_t spread_pair(uint32_t x)
{
    constexpr int perm = ODD ? 0xF5 : 0xA0;  // quad_perm [1,1,3,3] or [0,0,2,2]
    return __builtin_amdgcn_mov_dpp(x, perm, 0xF, 0xF, false);
}

template <int ODD>
__device__ inline float spread_pair(float x)
{
    return __builtin_bit_cast(float, spread_pair<ODD>(__builtin_bit_cast(uint32_t, x)));
}

template <int ODD>
__device__ inline double spread_pair(double x)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    return __builtin_bit_cast(double, (uint64_t)spread_pair<ODD>((uint32_t)u) |
                                          ((uint64_t)spread_pair<ODD>((uint32_t)(u >> 32)) << 32));
}

// right-hand sides of the least-squares systems of the three variables of layer l of cell c (training
// features): average differences, then scaled gradients of the cell and its face neighbours
template <typename R>
__device__ inline void recon_rhs(const MeshDev &m, const LayerW<R> *__restrict__ W, const LayerG<R> *__restrict__ G, int l,
                                 int64_t c, double &Q0h, R rhs[3][17])
{
    const int64_t T = m.T;
    const R hs = tab<R>(m.hs)[c];
    const LayerW<R> w0 = W[2 * c + l];
    Q0h = w0.h;
    int64_t nb[9];
#pragma unroll
    for (int s = 0; s < 9; s++) {
        nb[s] = GKS_IX(m.sten[s * T + c], T + m.NG);
        const LayerW<R> w = W[2 * nb[s] + l];
        // differences of thicknesses are taken in FP64 before rounding
        rhs[0][s] = (R)(w.h - w0.h);
        rhs[1][s] = w.m[0] - w0.m[0];
        rhs[2][s] = w.m[1] - w0.m[1];
    }
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const LayerG<R> g = G[2 * (k == 0 ? c : nb[k - 1]) + l];
#pragma unroll
        for (int q = 0; q < 3; q++) {
            rhs[q][9 + 2 * k] = hs * g.g[2 * q];
            rhs[q][10 + 2 * k] = hs * g.g[2 * q + 1];
        }
    }
}

// nothing is scheduled across this point: bounds what the scheduler holds in flight at once
__device__ inline void sched_fence() { __builtin_amdgcn_sched_barrier(0); }

// Makes the compiler treat the values as computed here and new: what they come from is not moved
// below this point, and what was computed from them before is formed again afterwards instead of
// being held in registers meanwhile.
template <typename R, int N>
__device__ inline void settle(R (&v)[N])
{
#pragma unroll
    for (int i = 0; i < N; i++) asm volatile("" : "+v"(v[i]));
}

// The reconstructions of the three variables of one layer (q = 0 the thickness, 1 and 2 the momenta)
// in scaled coordinates, as deviations from the cell averages:
//   ratio (P - mean) + sx x + sy y,  P = a0 x + a1 y + a2 x^2 + a3 xy + a4 y^2 + a5 x^3 + ... + a8 y^3
// In FP64 the combination is folded into the coefficients (ratio = 1, sx = sy = 0, not stored): fewer
// operations, and 18 registers less through the evaluation.  In FP32 it is not: the mixed path's rounding
// is amplified at a few obtuse cells of jittered meshes until the smoothness floor holds it (1e-5 of the
// variable), so that any other order of its FP32 operations gives gradients there that differ by as
// much; the order is kept, expression by expression.
template <typename R>
constexpr bool FOLD = sizeof(R) == 8;

template <typename R>
struct Fit {
    R a[3][9], mean[3];
    R ratio[3], sx[3], sy[3];
};

// products that are rounded before they are added (no fused multiply-add)
template <typename R>
__device__ inline R rounded(R a, R b)
{
#pragma clang fp contract(off)
    R p = a * b;
    asm volatile("" : "+v"(p));
    return p;
}

template <typename R>
__device__ inline R fit_dev(const Fit<R> &f, int q, R x, R y, bool first = false)
{
    const R *a = f.a[q];
    if constexpr (FOLD<R>) {
        const R xx = x * x, yy = y * y;
        return a[0] * x + a[1] * y + a[2] * xx + a[3] * (x * y) + a[4] * yy + (a[5] * x + a[6] * y) * xx +
               (a[7] * x + a[8] * y) * yy - f.mean[q];
    } else {
        const R P = a[0] * x + a[1] * y + a[2] * x * x + a[3] * x * y + a[4] * y * y + a[5] * x * x * x +
                    a[6] * x * x * y + a[7] * x * y * y + a[8] * y * y * y - f.mean[q];
        return first ? fma(f.sy[q], y, fma(f.ratio[q], P, rounded(f.sx[q], x)))
                     : fma(f.sy[q], y, fma(f.sx[q], x, rounded(f.ratio[q], P)));
    }
}

// derivatives of P; in scaled coordinates
template <typename R>
__device__ inline R fit_px(const R *a, R x, R y)
{
    if constexpr (FOLD<R>)
        return a[0] + a[2] * (2 * x) + a[3] * y + a[5] * (3 * (x * x)) + a[6] * (2 * x * y) + a[7] * (y * y);
    else
        return a[0] + 2 * a[2] * x + a[3] * y + 3 * a[5] * x * x + 2 * a[6] * x * y + a[7] * y * y;
}

template <typename R>
__device__ inline R fit_py(const R *a, R x, R y)
{
    if constexpr (FOLD<R>)
        return a[1] + a[3] * x + a[4] * (2 * y) + a[6] * (x * x) + a[7] * (2 * x * y) + a[8] * (3 * (y * y));
    else
        return a[1] + a[3] * x + 2 * a[4] * y + a[6] * x * x + 2 * a[7] * x * y + 3 * a[8] * y * y;
}

template <typename R>
__device__ inline R fit_dx(const Fit<R> &f, int q, R x, R y, R ihs)
{
    const R P = fit_px(f.a[q], x, y);
    if constexpr (FOLD<R>)
        return P * ihs;
    else
        return (f.ratio[q] * P + f.sx[q]) * ihs;
}

template <typename R>
__device__ inline R fit_dy(const Fit<R> &f, int q, R x, R y, R ihs)
{
    if constexpr (FOLD<R>) {
        return fit_py(f.a[q], x, y) * ihs;
    } else {
        const R *a = f.a[q];
        R P = fma(2 * a[4], y, a[1] + rounded(a[3], x)) + rounded(a[6] * x, x);
        P = fma(3 * a[8] * y, y, fma(2 * a[7] * x, y, P));
        return (f.ratio[q] * P + f.sy[q]) * ihs;
    }
}

// The nonlinear weights of a layer's three variables from their P^3 coefficients f.a and the
// differences that the plane candidates take, d[64 (5 q + i)], i = 0..2 to the face neighbours and 3, 4
// the scaled gradient; completes f and returns the thickness's weight ratio omega_0 / d_0.
template <typename R>
__device__ inline R recon_weights(const Phys &p, bool lin, unsigned cmask, const R *nbc, int64_t T, unsigned cl, double Q0h,
                                  double hl, const R Qm[2], const R vx[3], const R vy[3], const R *d, Fit<R> &f)
{
    // cell means of the basis (centroid at the origin)
    {
        R mxx = 0, mxy = 0, myy = 0, mx3 = 0, mx2y = 0, mxy2 = 0, my3 = 0;
#pragma unroll
        for (int k = 0; k < 3; k++) {
            mxx += vx[k] * vx[k];
            mxy += vx[k] * vy[k];
            myy += vy[k] * vy[k];
            mx3 += vx[k] * vx[k] * vx[k];
            mx2y += vx[k] * vx[k] * vy[k];
            mxy2 += vx[k] * vy[k] * vy[k];
            my3 += vy[k] * vy[k] * vy[k];
        }
        const R c12 = R(1) / R(12), c30 = R(1) / R(30);
#pragma unroll
        for (int q = 0; q < 3; q++) {
            const R *a = f.a[q];
            f.mean[q] = a[2] * mxx * c12 + a[3] * mxy * c12 + a[4] * myy * c12 + a[5] * mx3 * c30 + a[6] * mx2y * c30 +
                        a[7] * mxy2 * c30 + a[8] * my3 * c30;
        }
    }
    // lower-order candidates (reading of the nonlinear compact reconstruction): planes through
    // the averages of {0, f0, f1}, {0, f1, f2}, {0, f2, f0} and the cell's own gradient.  A
    // sub-stencil whose centroid offsets are nearly parallel is not a candidate (bit clear in
    // cmask, decided at setup in FP64): its plane would carry a huge slope into the combination
    // below; its linear weight goes to P^3.
    cmask |= 8u;  // the own-gradient plane is always a candidate
    const int ncand = __builtin_popcount(cmask);
    const R d0 = ncand == 4 ? R(0.8) : ncand == 3 ? R(0.85) : ncand == 2 ? R(0.9) : R(0.95), dm = R(0.05);
    const bool nonlinear = !p.linear && !lin;
    R beta0[3] = {0, 0, 0};
    if (nonlinear) {
        // smoothness indicator of P^3 in scaled coordinates: the cell has area 1/2 there, so the
        // |Omega|^(|alpha|-1) weights become (1/2)^(|alpha|-1) and integrals are averages / 2.
        // First derivatives (quadratics): 6-point degree-4 rule; second (linear): edge midpoints.
        const R qa[2] = {R(0.445948490915964886), R(0.091576213509770743)};
        const R qw[2] = {R(0.223381589678011466), R(1.0 / 3.0 - 0.223381589678011466)};
        R s1[3] = {0, 0, 0}, s2[3] = {0, 0, 0};
#pragma unroll
        for (int r = 0; r < 2; r++)
#pragma unroll
            for (int j = 0; j < 3; j++) {
                R x, y;
                if constexpr (FOLD<R>) {  // (1 - 2 qa) v_j + qa (v_i + v_k), with v_i + v_k = -v_j about the centroid
                    x = (1 - 3 * qa[r]) * vx[j];
                    y = (1 - 3 * qa[r]) * vy[j];
                } else {
                    const R l0 = (j == 0) ? 1 - 2 * qa[r] : qa[r];
                    const R l1 = (j == 1) ? 1 - 2 * qa[r] : qa[r];
                    const R l2 = (j == 2) ? 1 - 2 * qa[r] : qa[r];
                    x = l0 * vx[0] + l1 * vx[1] + l2 * vx[2];
                    y = l0 * vy[0] + l1 * vy[1] + l2 * vy[2];
                }
#pragma unroll
                for (int q = 0; q < 3; q++) {
                    const R px = fit_px(f.a[q], x, y), py = fit_py(f.a[q], x, y);
                    s1[q] += qw[r] * fma(px, px, rounded(py, py));
                }
                sched_fence();
            }
#pragma unroll
        for (int j = 0; j < 3; j++) {
            const R x = R(0.5) * (vx[j] + vx[(j + 1) % 3]), y = R(0.5) * (vy[j] + vy[(j + 1) % 3]);
#pragma unroll
            for (int q = 0; q < 3; q++) {
                const R *a = f.a[q];
                const R pxx = 2 * a[2] + 6 * a[5] * x + 2 * a[6] * y;
                const R pxy = a[3] + 2 * a[6] * x + 2 * a[7] * y;
                const R pyy = 2 * a[4] + 2 * a[7] * x + 6 * a[8] * y;
                s2[q] += fma(pyy, pyy, fma(pxx, pxx, rounded(pxy, pxy))) * (R(1) / R(3));
            }
            sched_fence();
        }
#pragma unroll
        for (int q = 0; q < 3; q++) {
            const R *a = f.a[q];
            const R s3 = fma(36 * a[8], a[8], fma(4 * a[7], a[7], fma(36 * a[5], a[5], rounded(4 * a[6], a[6]))));
            beta0[q] = R(0.5) * s1[q] + R(0.25) * s2[q] + R(0.125) * s3;
        }
    }
    R ox[3], oy[3], inv[3];
#pragma unroll
    for (int s = 0; s < 3; s++) {
        ox[s] = (nbc + (2 * s) * T)[cl];
        oy[s] = (nbc + (2 * s + 1) * T)[cl];
    }
#pragma unroll
    for (int s = 0; s < 3; s++) {
        const int sb = (s + 1) % 3;
        const R invd = R(1) / (ox[s] * oy[sb] - oy[s] * ox[sb]);
        inv[s] = ((cmask >> s) & 1u) ? invd : R(0);  // excluded planes: slope 0, weight 0
    }
    R ratio0 = 1;
#pragma unroll
    for (int q = 0; q < 3; q++) {
        R bx[4], by[4];
#pragma unroll
        for (int s = 0; s < 3; s++) {
            const int sb = (s + 1) % 3;
            const R ra = d[64 * (5 * q + s)], rb = d[64 * (5 * q + sb)];
            bx[s] = fma(ra, oy[sb], -rounded(oy[s], rb)) * inv[s];
            by[s] = fma(ox[s], rb, -rounded(ra, ox[sb])) * inv[s];
        }
        bx[3] = d[64 * (5 * q + 3)];
        by[3] = d[64 * (5 * q + 4)];
        R w0 = d0, wm[4];
#pragma unroll
        for (int s = 0; s < 4; s++) wm[s] = ((cmask >> s) & 1u) ? dm : R(0);
        // FP64: the planes' slopes weighted by their linear weights and by the nonlinear ones, in place
        // of the four weights
        R lx = 0, ly = 0, nx = 0, ny = 0;
        if constexpr (FOLD<R>) {
#pragma unroll
            for (int s = 0; s < 4; s++) {
                lx += wm[s] * bx[s];
                ly += wm[s] * by[s];
            }
            nx = lx;
            ny = ly;
        }
        if (nonlinear) {
            R tz = 0, bm[4];
#pragma unroll
            for (int s = 0; s < 4; s++) {
                bm[s] = R(0.5) * (s < 3 ? fma(bx[s], bx[s], rounded(by[s], by[s])) : fma(by[s], by[s], rounded(bx[s], bx[s])));
                tz += ((cmask >> s) & 1u) ? fabs(beta0[q] - bm[s]) : R(0);
            }
            if constexpr (FOLD<R>)
                tz *= ncand == 4 ? R(0.25) : ncand == 3 ? R(1.0 / 3.0) : ncand == 2 ? R(0.5) : R(1);
            else
                tz = ncand == 4 ? tz * R(0.25) : div_(tz, R(ncand));
            // floor of the smoothness indicators with the variable's scale: the level of a thickness,
            // 1e-8 h sqrt(G h) of the layer for a momentum
            const R Q0 = q == 0 ? (R)Q0h : Qm[q - 1];
            const R S2 = q == 0 ? R(1e-20) : (R)(1e-16 * p.G * hl * hl * hl);
            const R Q2 = fmax(Q0 * Q0, S2), epsw = rounded(eps_rel<R>(), Q2);
            const R t0 = d0 * (1 + div_(tz, fma(eps_rel<R>(), Q2, beta0[q])));
            R sum = t0, tm[4], sx = 0, sy = 0;
            // where every unnormalised weight equals its linear weight (tau = 0, or tau / (beta + eps)
            // below the rounding of 1), the weights are the linear ones, which sum to one: take them
            // exactly instead of dividing by their rounded sum
            bool same = t0 == d0;
#pragma unroll
            for (int s = 0; s < 4; s++) {
                tm[s] = ((cmask >> s) & 1u) ? dm * (1 + div_(tz, bm[s] + epsw)) : R(0);
                sum += tm[s];
                same = same && tm[s] == wm[s];
                if constexpr (FOLD<R>) {
                    sx += tm[s] * bx[s];
                    sy += tm[s] * by[s];
                    if (s & 1) sched_fence();
                }
            }
            const R isum = same ? R(1) : div_(R(1), sum);
            w0 = t0 * isum;
            if constexpr (FOLD<R>) {
                nx = sx * isum;
                ny = sy * isum;
            } else {
#pragma unroll
                for (int s = 0; s < 4; s++) wm[s] = tm[s] * isum;
            }
        }
        const R ratio = w0 / d0;
        if (q == 0) ratio0 = ratio;
        // combined polynomial R = ratio (P0 - sum dm Pm) + sum wm Pm, Pm = Q0 + b . x; all candidates
        // share the cell average Q0 (the weights sum to one)
        R sbx = 0, sby = 0;
        if constexpr (FOLD<R>) {
            sbx = nx - ratio * lx;
            sby = ny - ratio * ly;
            f.a[q][0] = ratio * f.a[q][0] + sbx;
            f.a[q][1] = ratio * f.a[q][1] + sby;
#pragma unroll
            for (int i = 2; i < 9; i++) f.a[q][i] *= ratio;
            f.mean[q] *= ratio;
        } else {
#pragma unroll
            for (int s = 0; s < 4; s++) {
                const R cm = wm[s] - ratio * (((cmask >> s) & 1u) ? dm : R(0));
                sbx += cm * bx[s];
                sby += cm * by[s];
            }
            f.ratio[q] = ratio;
            f.sx[q] = sbx;
            f.sy[q] = sby;
        }
        sched_fence();
    }
    return ratio0;
}

// the learned indicator inside the reconstruction: bf16 weight matrices, FP32 parameters, logit
// threshold, and where to leave the decisions (1 = linear weights) for inspection
struct IndArgs {
    const short *W1b, *W2b;
    const float *P;
    float thr;
    uint8_t *mask;
};

// whether cell c lies in the front band of the upper layer (h2) or the lower (eta1 - B); a wall ghost
// holds its cell's mirrored state and bottom
template <typename R>
__device__ inline bool wd_band(const MeshDev &m, const Phys &p, const LayerW<R> *__restrict__ W, bool lower, int64_t c)
{
    const int64_t T = m.T, TG = m.T + m.NG;
    double hk[4];
#pragma unroll
    for (int l = 0; l < 4; l++) {
        const int64_t i = l == 0 ? c : (int64_t)GKS_IX(m.sten[(l - 1) * T + c], TG);
        double h = W[2 * i + (lower ? 1 : 0)].h;
        if (lower) h -= m.Bbar[i < T ? i : (int64_t)GKS_IX(m.gsrc[i - T], T)];
        hk[l] = h;
    }
    const double hmax = fmax(fmax(hk[0], hk[1]), fmax(hk[2], hk[3])), thin = WD_THIN * p.h_dry;
    bool band = false;
#pragma unroll
    for (int l = 0; l < 4; l++) band = band || hk[l] < thin || hk[l] < WD_FRONT * hmax;
    // the lower layer thinner than the bottom's rise across the cell (scale sqrt(2 area)): its
    // shoreline lies inside the cell (a partially flooded cell)
    if (lower) {
        const double gx = m.gB[c], gy = m.gB[T + c];
        band = band || hk[0] < sqrt(2.0 * m.area[c]) * sqrt(gx * gx + gy * gy);
    }
    return band;
}

// One wave takes the 32 cells of a block of operators; a lane holds all three variables of its layer.
//
// On large meshes bound by memory: 520k cells FP64 move 1.29 GB a launch at the rate of a large copy, of
// which the operators' stream is half (1,248 bytes a cell; 624 in FP32).  On small ones by the rate of
// issue and the latency of the scattered reads along one wave's chain.  The 27 coefficients a lane keeps
// allow three waves a SIMD in FP64 (168 registers; where the indicator is evaluated two, 174: its two
// stages take 272 us on average at 520k cells, 299 before) and four in FP32.
// Before, with the state as one array a variable, 15 scattered 8-byte reads a stencil cell kept the address
// units 78 % busy, and the operators, staged by a block through LDS behind barriers, the reads, the
// arithmetic and the records ran one after another (taking any of them out shortened the kernel by its own
// time).  Hence a layer's averages and gradients each in one piece (one wide read a stencil cell), a wave
// to itself whose barriers are no instructions, the operators read straight into registers eight loads
// ahead and shared between a cell's two lanes by DPP, and the records turned in LDS into whole lines.
// 520k cells, between events: FP64 285 us before, 228 after; FP32 148, 128; 80k cells FP64 47.7, 39.8.  At
// 800 cells one wave's chain is all there is, 11.4 before, 13.6 after; 20 loads ahead instead of eight
// leave that and all sizes unchanged or slower (80k 46.5).
// IND: the learned indicator decides per cell whether the smoothness indicators are computed.
// IND = 1: its 44 features come from the right-hand sides the wave has gathered anyway; the wave
// evaluates the network for its 32 cells on the matrix cores and the decisions go to ind.mask.
// IND = 2: the decisions are read from ind.mask (the network ran on the step's first stage, the
// second reuses them).
// SRC = 1: the higher-order layer coupling (Sec. 3.2, Eq. SWE-source-discretization, and its remark
// that more integration points raise the order): the part of the cell average of h_a grad h_b that
// the product of averages misses, mean((h_a - mean h_a) grad h_b), and its time derivative with the
// thickness rate h_t = -div(h U), from the cell's own reconstructions, into src[8][T].  Radon's
// 7-point rule is exact for these degree-5 products; the two layers of a cell exchange their
// gradients between their two lanes.
// WD = 1: wet/dry layers (Phys::h_dry > 0), the front band's first-order reconstruction; it excludes
// the indicator and the higher-order coupling (the library rejects the combinations).
template <typename R, int IND, int SRC = 0, int WD = 0>
__global__ void __launch_bounds__(64, (sizeof(R) == 8 ? 3 : 4)) k_recon(MeshDev m, Phys p, const LayerW<R> *__restrict__ W,
                                              const LayerG<R> *__restrict__ G, IndArgs ind, GpRecs<R> rec,
                                              R *__restrict__ r0, R *__restrict__ src)
{
    // LDS: the differences that the plane candidates take, put away here while the fit needs the
    // registers; then, in the same space, the records of one local edge (two points) of the 32 cells,
    // heads then tails, each cell's span padded by 8 bytes so that the lanes' 8-byte writes fall on
    // different banks.  The indicator's features lie behind the differences, and behind those the
    // thickness's right-hand side until the features are made of it, then the hidden activations.
    constexpr int HB2 = 2 * (int)sizeof(GpHead<R>), TB2 = 2 * (int)sizeof(GpTail<R>);
    constexpr int HS = HB2 + 8, TS = TB2 + 8;
    constexpr int OBYTES = RECON_CELLS * (HS + TS), DBYTES = 15 * 64 * (int)sizeof(R);
    constexpr int FBYTES = RECON_CELLS * FB * 2, QBYTES = 17 * 64 * (int)sizeof(R), ABYTES = RECON_CELLS * (HB * 2 + 1);
    constexpr int IBYTES = DBYTES + (IND == 1 ? FBYTES + (QBYTES > ABYTES ? QBYTES : ABYTES) : 0);
    __shared__ uint4 lds[((OBYTES > IBYTES ? OBYTES : IBYTES) + 15) / 16];
    typedef R R2 __attribute__((ext_vector_type(2)));
    const int lane = threadIdx.x >> 1, l = threadIdx.x & 1;
    const bool lower = l == 1;
    const int64_t T = m.T, TG = m.T + m.NG;
    const int64_t blk = xcd_block(), c0 = blk * RECON_CELLS;
    const int ncell = T - c0 < RECON_CELLS ? (int)(T - c0) : RECON_CELLS;
    const bool valid = lane < ncell;
    // lanes beyond the last cell take its state and tables with the zeros that pad the operators, and write
    // nothing; a wave's cells lie at a uniform base plus a small index, so that the tables' addresses stay
    // in scalar registers
    const unsigned cl = (valid ? lane : ncell - 1) & (RECON_CELLS - 1);
    const int64_t c = c0 + cl;
    int32_t nb[9];
#pragma unroll
    for (int s = 0; s < 9; s++) nb[s] = GKS_IX((m.sten + s * T + c0)[cl], TG);
    const R hs = (tab<R>(m.hs) + c0)[cl];
    const LayerW<R> *Wl = W + l;
    const LayerG<R> *Gl = G + l;
    const LayerW<R> w0 = (W + 2 * c0)[2 * cl + l];
    const double Q0h = w0.h, hl = lower ? Q0h - (m.Bbar + c0)[cl] : Q0h;
    const R Qm[2] = {w0.m[0], w0.m[1]};
    // made here, before the fit, the test holds one bit and not the stencil's addresses through it
    const bool band = WD && wd_band(m, p, W, lower, c);
    // P^3 coefficients: the operator's column r times the right-hand side's entry r of each variable
    Fit<R> f;
    auto &a = f.a;
    R *d = reinterpret_cast<R *>(lds) + threadIdx.x;
    R *rh = reinterpret_cast<R *>(reinterpret_cast<char *>(lds) + DBYTES + FBYTES) + threadIdx.x;
    double td = 0, md = 0;  // largest differences of the thickness and of the momenta (features)
    {
        // Software pipeline: the operator's loads run AHEAD loads in front of their use and the gathers
        // of an entry RHS_AHEAD entries in front; the scheduling fences keep the compiler from sinking
        // them to their uses (a handful of loads in flight per wave instead of AHEAD + 3 RHS_AHEAD).
        constexpr int AHEAD = 8, RHS_AHEAD = 3;
        const R2 *M = reinterpret_cast<const R2 *>(m.M) + blk * (OP_LOADS * 64) + threadIdx.x;
        R2 ring[AHEAD];
#pragma unroll
        for (int j = 0; j < AHEAD; j++) ring[j] = M[64 * j];
        // what a stencil cell contributes: its averages (entries 0 to 8), or the gradients of the cell and
        // its face neighbours (two entries each, 9 to 16)
        LayerW<R> wq[RHS_AHEAD];
        LayerG<R> gq[2];
#pragma unroll
        for (int s = 0; s < RHS_AHEAD; s++) wq[s] = Wl[2 * (int64_t)nb[s]];
        R row[4];  // operator entries 4 j .. 4 j + 3 of the lane's cell
#pragma unroll
        for (int r = 0; r < 17; r++) {
            R b[3];
            if (r < 9) {
                const LayerW<R> w = wq[r % RHS_AHEAD];
                // differences of thicknesses are taken in FP64 before rounding
                b[0] = (R)(w.h - Q0h);
                b[1] = w.m[0] - Qm[0];
                b[2] = w.m[1] - Qm[1];
                if constexpr (IND == 1) {
                    td = fmax(td, fabs((double)b[0]));
                    md = fmax(md, fmax(fabs((double)b[1]), fabs((double)b[2])));
                }
                if (r + RHS_AHEAD < 9) wq[r % RHS_AHEAD] = Wl[2 * (int64_t)nb[r + RHS_AHEAD]];
                if (r == 5) gq[0] = (G + 2 * c0)[2 * cl + l];
                if (r == 7) gq[1] = Gl[2 * (int64_t)nb[0]];
            } else {
                const int k = (r - 9) / 2;
#pragma unroll
                for (int q = 0; q < 3; q++) b[q] = hs * gq[k & 1].g[2 * q + ((r - 9) & 1)];
                if ((r == 10 || r == 12) && k < 2) gq[k & 1] = Gl[2 * (int64_t)nb[k + 1]];
            }
            if (r < 3 || r == 9 || r == 10) {
#pragma unroll
                for (int q = 0; q < 3; q++) d[64 * (5 * q + (r < 3 ? r : r - 6))] = b[q];
            }
            if constexpr (IND == 1) rh[64 * r] = b[0];
#pragma unroll
            for (int i = 0; i < 9; i++) {
                const int e = 9 * r + i, j = e / 4;
                if (e % 4 == 0) {
                    const R2 v = ring[j % AHEAD];
                    row[0] = spread_pair<0>((R)v[0]);
                    row[1] = spread_pair<0>((R)v[1]);
                    row[2] = spread_pair<1>((R)v[0]);
                    row[3] = spread_pair<1>((R)v[1]);
                    if (j + AHEAD < OP_LOADS) ring[j % AHEAD] = M[64 * (j + AHEAD)];
                    sched_fence();
                }
#pragma unroll
                for (int q = 0; q < 3; q++) a[q][i] = r == 0 ? row[e % 4] * b[q] : fma(row[e % 4], b[q], a[q][i]);
            }
        }
    }
#pragma unroll
    for (int q = 0; q < 3; q++) settle(a[q]);
    bool lin = false;
    if constexpr (IND == 2) lin = (ind.mask + c0)[cl] != 0;
    if constexpr (IND == 1) {
        short(*feat)[FB] = reinterpret_cast<short(*)[FB]>(reinterpret_cast<char *>(lds) + DBYTES);
        short(*hid)[HB] = reinterpret_cast<short(*)[HB]>(&feat[RECON_CELLS][0]);
        uint8_t *skip = reinterpret_cast<uint8_t *>(&hid[RECON_CELLS][0]);
        const int fl = lower ? 0 : 1;
        {
            const double s = td + 1e-12 * fabs(Q0h), is = 1.0 / s;
#pragma unroll
            for (int k = 0; k < 17; k++) feat[lane][17 * fl + k] = to_bf16(thick_feature((double)rh[64 * k], is));
            feat[lane][34 + fl] = to_bf16(size_feature(s, hl));
        }
        feat[lane][36 + fl] = to_bf16(mom_feature(md, hl, p.G));
        if (lower) {
#pragma unroll
            for (int k = 0; k < 6; k++) feat[lane][38 + k] = to_bf16((m.igeo + k * T + c0)[cl]);
        } else {
#pragma unroll
            for (int k = MLP_IN; k < MLP_K; k++) feat[lane][k] = 0;
        }
        __syncthreads();
        mlp_layer1(feat, hid, threadIdx.x, 0, ind.W1b, ind.P);
        sched_fence();
        mlp_layer1(feat, hid, threadIdx.x, 1, ind.W1b, ind.P);
        __syncthreads();
        sched_fence();
        float z[16];
        mlp_layer2_out(hid, threadIdx.x, ind.W2b, ind.P, z);
        sched_fence();
        if ((threadIdx.x & 31) == 0) {
            const int half = threadIdx.x >> 5;
#pragma unroll
            for (int r = 0; r < 16; r++) skip[8 * (r / 4) + 4 * half + (r % 4)] = z[r] > ind.thr ? 1 : 0;
        }
        __syncthreads();
        lin = skip[lane] != 0;
        if (lower && valid) ind.mask[c] = lin ? 1 : 0;
    }
    // scaled vertices (centroid at the origin)
    const R *vt = tab<R>(m.vtx) + c0;
    R vx[3], vy[3];
#pragma unroll
    for (int k = 0; k < 3; k++) {
        vx[k] = (vt + (2 * k) * T)[cl];
        vy[k] = (vt + (2 * k + 1) * T)[cl];
    }
    R ratio = recon_weights<R>(p, lin, (m.cand + c0)[cl], tab<R>(m.nbc) + c0, T, cl, Q0h, hl, Qm, vx, vy, d, f);
    const R ihs = div_(R(1), hs);
    const double gB[2] = {lower ? (m.gB + c0)[cl] : 0.0, lower ? (m.gB + T + c0)[cl] : 0.0};
    const R gs[2] = {R(0.5 - 0.28867513459481288225), R(0.5 + 0.28867513459481288225)};
    double h6[6];  // the thickness at the Gauss points
    R theta = 1;
    {
        // positivity safeguard (not in the paper): where a layer thickness at a Gauss point would fall
        // below a tenth of the cell's average, the deviation from the average is scaled down
        // (Zhang-Shu scaling) until it does not; the lower layer's thickness is eta1 minus the
        // piecewise-linear bottom.  The factor is 1 at rest and in ordinary flows; it is formed in the
        // bulk precision (it only decides how far to pull the values back).
        const R hbar = (R)hl, floor_h = R(0.1) * hbar;
        const R gBx = (R)gB[0], gBy = (R)gB[1];
#pragma unroll
        for (int slot = 0; slot < 6; slot++) {
            const int k = slot / 2, k1 = (k + 1) % 3, g = slot & 1;
            const R x = vx[k] + gs[g] * (vx[k1] - vx[k]);
            const R y = vy[k] + gs[g] * (vy[k1] - vy[k]);
            const R dev = fit_dev(f, 0, x, y, slot == 0);
            h6[slot] = Q0h + (double)dev;
            if (dev < 0) {
                const R bdev = hs * (gBx * x + gBy * y), room = hbar - bdev - floor_h;
                // FP64: a quotient of at least 1 changes nothing and is not formed
                if (!FOLD<R> || room < -dev) theta = fmin(theta, fmax(R(0), div_(room, -dev)));
            }
            sched_fence();
        }
        if (theta < R(1)) {
#pragma unroll
            for (int slot = 0; slot < 6; slot++) h6[slot] = Q0h + (double)theta * (h6[slot] - Q0h);
        }
    }
    R Qv[2] = {Qm[0], Qm[1]};
    if (WD && band) {
        // front band: the layer's cell average, thickness constant (the lower layer's level follows
        // the bottom), momentum the thickness times the desingularised velocity; r0 = 0 marks it
#pragma unroll
        for (int q = 0; q < 2; q++) Qv[q] = (R)(hl * wd_velocity(hl, (double)Qm[q], p.h_dry));
#pragma unroll
        for (int slot = 0; slot < 6; slot++) {
            const int k = slot / 2, k1 = (k + 1) % 3, g = slot & 1;
            const R x = vx[k] + gs[g] * (vx[k1] - vx[k]);
            const R y = vy[k] + gs[g] * (vy[k1] - vy[k]);
            h6[slot] = fma((double)hs, fma(gB[1], (double)y, rounded(gB[0], (double)x)), Q0h);
        }
        ratio = R(0);
    }
    if (valid) (r0 + c0)[(lower ? 0 : T) + cl] = ratio;
    // the records, one local edge (two points) at a time through LDS; the points' monomials are formed
    // again and not kept from above (60 registers in FP64).  They lie over other lanes' differences, which
    // have to be read before: the block is one wave, so the barrier is an order for the compiler and no
    // instruction
    __syncthreads();
    settle(vx);
    settle(vy);
    char *lh = reinterpret_cast<char *>(lds) + lane * HS, *lt = reinterpret_cast<char *>(lds) + RECON_CELLS * HS + lane * TS;
#pragma unroll
    for (int k = 0; k < 3; k++) {
#pragma unroll
        for (int g = 0; g < 2; g++) {
            const int k1 = (k + 1) % 3;
            const R x = vx[k] + gs[g] * (vx[k1] - vx[k]);
            const R y = vy[k] + gs[g] * (vy[k1] - vy[k]);
            char *h = lh + g * (int)sizeof(GpHead<R>), *t = lt + g * (int)sizeof(GpTail<R>) + (lower ? 6 : 0) * (int)sizeof(R);
            *reinterpret_cast<double *>(h + (lower ? 8 : 0)) = h6[2 * k + g];
            R *hm = reinterpret_cast<R *>(h + 16) + (lower ? 2 : 0), *gt = reinterpret_cast<R *>(t);
#pragma unroll
            for (int q = 1; q < 3; q++) {
                const R dev = fit_dev(f, q, x, y, k == 0 && g == 0);
                hm[q - 1] = WD && band ? Qv[q - 1] : Qv[q - 1] + dev;
            }
#pragma unroll
            for (int q = 0; q < 3; q++) {
                R gx = fit_dx(f, q, x, y, ihs), gy = fit_dy(f, q, x, y, ihs);
                if (q == 0 && theta < R(1)) {
                    gx *= theta;
                    gy *= theta;
                }
                if (WD && band) {
                    gx = q == 0 ? (R)gB[0] : R(0);
                    gy = q == 0 ? (R)gB[1] : R(0);
                }
                gt[2 * q] = gx;
                gt[2 * q + 1] = gy;
                sched_fence();
            }
        }
        __syncthreads();
        // copy out: the block's span of this edge, 16-byte words
        struct alignas(8) W16 {
            uint64_t a, b;
        };
        constexpr int HW = HB2 / 16, TW = TB2 / 16;
        const char *l0 = reinterpret_cast<const char *>(lds);
        uint4 *oh = reinterpret_cast<uint4 *>(rec.head + rec_at(T, c0, k, 0)), *ot = reinterpret_cast<uint4 *>(rec.tail + rec_at(T, c0, k, 0));
#pragma unroll
        for (int j = 0; j < RECON_CELLS * HW / 64; j++) {
            const int i = threadIdx.x + 64 * j;
            const W16 w = *reinterpret_cast<const W16 *>(l0 + (i / HW) * HS + (i % HW) * 16);
            if (i < ncell * HW) oh[i] = __builtin_bit_cast(uint4, w);
        }
#pragma unroll
        for (int j = 0; j < RECON_CELLS * TW / 64; j++) {
            const int i = threadIdx.x + 64 * j;
            const W16 w = *reinterpret_cast<const W16 *>(l0 + RECON_CELLS * HS + (i / TW) * TS + (i % TW) * 16);
            if (i < ncell * TW) ot[i] = __builtin_bit_cast(uint4, w);
        }
        __syncthreads();
    }
    if constexpr (SRC == 1) {
        // Radon's 7-point rule (degree 5): the centroid, then two orbits (b, a, a) of barycentrics
        const R A1 = R(0.101286507323456338800987361915), B1 = R(0.797426985353087322398025276170);
        const R A2 = R(0.470142064105115089770441209513), B2 = R(0.059715871789769820459117580973);
        const R W0 = R(0.225), W1 = R(0.125939180544827152595683945500), W2 = R(0.132394152788506180737649387833);
        settle(vx);
        settle(vy);
        R gb2[2] = {0, 0}, f2[2] = {0, 0}, tg[2] = {0, 0}, ft[2] = {0, 0}, tm = 0;
        const R gBx = (R)gB[0], gBy = (R)gB[1], i2 = ihs * ihs;
        // kept rolled: unrolled, the points' common factors of the coefficients fill the registers
#pragma unroll 1
        for (int qi = 0; qi < 7; qi++) {
            R l0, l1, l2;
            if (qi == 0) {
                l0 = l1 = l2 = R(1) / R(3);
            } else if (qi <= 3) {
                l0 = qi == 1 ? B1 : A1;
                l1 = qi == 2 ? B1 : A1;
                l2 = qi == 3 ? B1 : A1;
            } else {
                l0 = qi == 4 ? B2 : A2;
                l1 = qi == 5 ? B2 : A2;
                l2 = qi == 6 ? B2 : A2;
            }
            const R x = l0 * vx[0] + l1 * vx[1] + l2 * vx[2];
            const R y = l0 * vy[0] + l1 * vy[1] + l2 * vy[2];
            const R wq = qi == 0 ? W0 : qi <= 3 ? W1 : W2;
            // own thickness: deviation and gradient (the lower layer's thickness is eta1 minus the bottom)
            R h = theta * fit_dev(f, 0, x, y), gx = fit_px(a[0], x, y), gy = fit_py(a[0], x, y);
            if constexpr (!FOLD<R>) {
                gx = f.ratio[0] * gx + f.sx[0];
                gy = f.ratio[0] * gy + f.sy[0];
            }
            gx = fma(theta * gx, ihs, -gBx);
            gy = fma(theta * gy, ihs, -gBy);
            if (lower) h -= hs * (gBx * x + gBy * y);
            // own thickness rate -div(h U) and its gradient: x-momentum's d/dx, y-momentum's d/dy
            const R c1 = FOLD<R> ? R(1) : f.ratio[1], c2 = FOLD<R> ? R(1) : f.ratio[2];
            const R uxx = 2 * a[1][2] + 6 * a[1][5] * x + 2 * a[1][6] * y, uxy = a[1][3] + 2 * a[1][6] * x + 2 * a[1][7] * y;
            const R vxy = a[2][3] + 2 * a[2][6] * x + 2 * a[2][7] * y, vyy = 2 * a[2][4] + 2 * a[2][7] * x + 6 * a[2][8] * y;
            const R s1 = FOLD<R> ? R(0) : f.sx[1], s2 = FOLD<R> ? R(0) : f.sy[2];
            R u[6] = {(c1 * fit_px(a[1], x, y) + s1) * ihs, (c2 * fit_py(a[2], x, y) + s2) * ihs,
                      c1 * uxx * i2, c2 * vxy * i2, c1 * uxy * i2, c2 * vyy * i2};
            settle(u);  // each rounded before the sums
            const R tau = -(u[0] + u[1]), tx = -(u[2] + u[3]), ty = -(u[4] + u[5]);
            // the other layer's gradients
            const R bx = __shfl_xor(gx, 1), by = __shfl_xor(gy, 1), btx = __shfl_xor(tx, 1), bty = __shfl_xor(ty, 1);
            f2[0] += wq * h * bx;
            f2[1] += wq * h * by;
            tg[0] += wq * tau * bx;
            tg[1] += wq * tau * by;
            gb2[0] += wq * bx;
            gb2[1] += wq * by;
            tm += wq * tau;
            ft[0] += wq * h * btx;
            ft[1] += wq * h * bty;
            sched_fence();
        }
        if (valid) {
            // rows 0, 1: lower (h1 - mean) grad h2; 2, 3: upper (h2 - mean) grad h1; 4..7 their rates,
            // sum w (tau_a - mean tau_a) grad h_b + sum w (h_a - mean) grad tau_b
            const int o = lower ? 0 : 2;
#pragma unroll
            for (int i = 0; i < 2; i++) {
                src[(o + i) * T + c] = f2[i];
                src[(4 + o + i) * T + c] = tg[i] - tm * gb2[i] + ft[i];
            }
        }
    }
}

// a b + k with the constant k in scalar registers (the compiler would copy it to vector registers with
// two moves an operation)
__host__ __device__ inline double fma_k(double a, double b, double k)
{
#ifdef __HIP_DEVICE_COMPILE__
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(k));
    return r;
#else
    return fma(a, b, k);
#endif
}

// 1/2 erfc(-x) of k_plane.  FP64: for -1/2 <= x <= 1, where almost all flows are, 1/2 + erf(x) / 2 with
// erf(x) = x + x P(x^2), P interpolated at the Chebyshev nodes (4e-17 of P).  Beyond, the library's erfc:
// below -1/2 the sum would lose the small fraction's digits (8e-16 of it at -1, 4e-9 at -4, all at -6).
// FP32 has the library's throughout: another last bit, once in 1e9 values, would show in the mixed
// path's results (Fit).
template <typename R>
__host__ __device__ inline double kinetic_fraction(double x)
{
    if constexpr (sizeof(R) == 4) return 0.5 * erfc(-x);
    if (!(x >= -0.5 && x <= 1.0)) return 0.5 * erfc(-x);
    const double s = x * x;
    double p = fma_k(s, -7.795898827002142e-10, 1.3720064546777686e-08);
    p = fma_k(p, s, -1.6208483801871705e-07);
    p = fma_k(p, s, 1.6447424703317362e-06);
    p = fma_k(p, s, -1.492473690741966e-05);
    p = fma_k(p, s, 0.00012055294904839707);
    p = fma_k(p, s, -0.0008548325975389692);
    p = fma_k(p, s, 0.0052239776071164225);
    p = fma_k(p, s, -0.02686617064323777);
    p = fma_k(p, s, 0.11283791670945006);
    p = fma_k(p, s, -0.37612638903183543);
    p = fma_k(p, s, 0.12837916709551256);
    return 0.5 + 0.5 * fma(x, p, x);
}

// --------------------------------------------------------------------------------------------
// time step

// a layer's |U| + sqrt(G h); the velocity is desingularised in a thin layer (wet/dry; m / h otherwise)
// and a dry cell may hold -0
template <typename R>
__device__ inline double wave_speed(const Phys &p, double h, const R *mom)
{
    const double u = wd_velocity(h, mom[0], p.h_dry), v = wd_velocity(h, mom[1], p.h_dry);
    return sqrt(fma2(u, u, v, v)) + sqrt(p.G * fmax(h, 0.0));
}

// One wave's part of the maxima; a NaN (a state gone bad) does not count.  A whole wave inside one
// scenario stores its maximum; with one atomic a wave instead, the second update of 180k cells FP32 took
// 45 us for 22.
// A wave with a border or with lanes outside the mesh sends atomics, lane by lane.
__device__ inline void max_speed(const Phys &p, int64_t wave, int sc, double v)
{
    v = fmax(v, 0.0);
    const bool whole = __ballot(sc == __builtin_amdgcn_readfirstlane(sc)) == ~0ull;
    if (whole) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off));
    } else {
        const unsigned long long bits = __builtin_bit_cast(unsigned long long, v);
        if (bits > __hip_atomic_load(p.smax + sc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(p.smax + sc, bits);
        v = 0;
    }
    if (__lane_id() == 0) p.speed[wave] = v;
}

__global__ void __launch_bounds__(256) k_clear(unsigned long long *__restrict__ x, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = 0;
}

// the maxima of a state that did not come from a step (smax holds zeros)
template <typename R>
__global__ void __launch_bounds__(256) k_speed(MeshDev m, Phys p, const LayerW<R> *__restrict__ W)
{
    const int64_t idx = xcd_block() * blockDim.x + threadIdx.x, c = idx >> 1;
    const int l = idx & 1;
    if (c >= m.T) return;
    const LayerW<R> w = W[2 * c + l];
    max_speed(p, idx >> 6, m.cscen ? (int)GKS_IX(m.cscen[c], m.S) : 0, wave_speed(p, l ? w.h - m.Bbar[c] : w.h, w.m));
}

__device__ inline void set_step(const MeshDev &m, const Phys &p, int s, double smax)
{
    double dt = p.cfl * m.sdxmin[s] / smax;
    const double t = p.scal[2 * s + 1];
    double tn = t + dt;
    if (tn > p.t_end[s]) {  // the last step ends exactly at t_end; none ever goes back
        dt = fmax(0.0, p.t_end[s] - t);
        tn = fmax(t, p.t_end[s]);
    }
    p.scal[2 * s] = dt;
    p.scal[2 * s + 1] = tn;
}

// what a launch of k_plane does for the step besides the planes
enum { STEP_NONE = 0, STEP_CFL = 1, STEP_GIVEN = 2 };

__host__ __device__ inline unsigned step_blocks(int S) { return (unsigned)(S + N_XCD - 1) / N_XCD * N_XCD; }

// one block: the step size of scenario s (STEP_CFL); its part of smax is cleared for the next update
__device__ inline void begin_step(const MeshDev &m, const Phys &p, int step, int s)
{
    __shared__ double sh[4];
    if (step == STEP_CFL) {
        // the waves whose first cell is the scenario's
        const int64_t w0 = (m.scell[s] + 31) / 32, w1 = (m.scell[s + 1] + 31) / 32;
        double v = __builtin_bit_cast(double, p.smax[s]);
        for (int64_t w = w0 + threadIdx.x; w < w1; w += 8 * blockDim.x) {
            double x[8];
#pragma unroll
            for (int i = 0; i < 8; i++) x[i] = w + i * blockDim.x < w1 ? p.speed[w + i * blockDim.x] : 0.0;
#pragma unroll
            for (int i = 0; i < 8; i++) v = fmax(v, x[i]);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off));
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int i = 1; i < (int)(blockDim.x >> 6); i++) v = fmax(v, sh[i]);
            set_step(m, p, s, v);
        }
    }
    if (threadIdx.x == 0) p.smax[s] = 0;
}

// --------------------------------------------------------------------------------------------
// interface force modelling (Sec. 2.3): gradient of the plane through the edge-centre heights of eta1
// (lower-layer velocity) and of h2 (upper-layer velocity), each from the two Gauss points' convex
// combinations (FP64: cheap, and the plane through them must be flat at rest)

// Only cells whose plane gradient the flux can read: the force model blends it in with weight 1 - w,
// w = min(1, omega0/d0 of both sides) taken as 1 within 1e-12 of it, so only next to a cell whose
// weight ratio is below 1 - 1e-12.  A face neighbour beyond a wall is the cell's own mirror image.
//
// Four lanes a cell, one for each Gauss point of an edge (bit 0) and field (bit 1), over the three edges;
// Green-Gauss, exact for planes.  Bound by latency: a chain of dependent reads (stencil, weights; edge,
// cells, records) and the error function.  An edge between two such cells is evaluated for both of them,
// which costs less than the heights' way through memory and two more launches: between events, three
// kernels (weights to a mark per cell, heights per edge, planes per cell) took 18.7 us a stage at 800
// cells FP64 where this one takes 9.5, 20.3 / 11.6 at 80k, 34.2 / 27.0 at 520k.
// Reading all three edges before the first is used and the short error function: 800 cells 6.9 -> 5.5 us a
// launch (in a trace), 10k 7.9 -> 5.7, 160k wet/dry 28.8 -> 24.7; 20k FP32, the reading alone, 9.0 -> 8.1.
//
// In a step's first stage one more block per scenario sets the step size from the largest wave speeds
// (nothing reads it before the fluxes).  As two kernels of their own over the state, the step sizes cost
// 5.2 us a step at 800 cells FP64, 13.3 us at 520k, 17.7 us at a million, 19.3 us on an ensemble of 12
// scenarios; here 2 to 9 us, most of it beside the planes (a million cells: 34.8 -> 38.8 us a launch).
template <typename R>
__global__ void __launch_bounds__(256) k_plane(MeshDev m, Phys p, int step, const GpHead<R> *__restrict__ head,
                                               const R *__restrict__ r0, double *__restrict__ gP1)
{
    // those blocks come first, for they take longest, and in eights, so that the others keep their XCDs
    const unsigned extra = step == STEP_NONE ? 0 : step_blocks(m.S);
    if (blockIdx.x < extra) {
        if ((int)blockIdx.x < m.S) begin_step(m, p, step, blockIdx.x);
        return;
    }
    const int64_t idx = xcd_block(extra) * blockDim.x + threadIdx.x, c = idx >> 2;
    if (c >= m.T) return;  // the lanes of a cell leave together, here and below
    const int j = idx & 3, g = j & 1, f = j >> 1;
    const int64_t T = m.T, E = m.E;
    // lane 0 looks at the cell's own weights, the others at a face neighbour's
    const int64_t i = j == 0 ? c : (int64_t)GKS_IX(m.sten[(j - 1) * T + c], T + m.NG);
    int need = i < T && ((double)r0[i] < W_ONE || (double)r0[T + i] < W_ONE);
    need |= __shfl_xor(need, 1);
    need |= __shfl_xor(need, 2);
    if (!need) return;
    // field 0: eta1 with the lower layer's momentum; 1: h2 with the upper layer's
    const int hq = f == 0 ? 1 : 0, mq = f == 0 ? 2 : 0;
    const R *en = tab<R>(m.en);
    // all three edges' reads are under way before any is used: a branch at the first (a wall, the error
    // function) would hold back the others'
    int64_t e[3];
    int32_t L[3], Rc[3], sl[3];
#pragma unroll
    for (int k = 0; k < 3; k++) {
        const int32_t code = m.cedge[k * T + c];
        e[k] = GKS_IX(code >= 0 ? code : ~code, E);
    }
#pragma unroll
    for (int k = 0; k < 3; k++) {
        L[k] = GKS_IX(m.eL[e[k]], T);
        Rc[k] = m.eR[e[k]] >= 0 ? GKS_IX(m.eR[e[k]], T) : m.eR[e[k]];
        sl[k] = m.eslot[e[k]];
    }
    double geo[3][5], z[3][2];  // normal, bottom, Green-Gauss weights; the sides' levels
    R q[3][4];                  // their momenta
#pragma unroll
    for (int k = 0; k < 3; k++) {
        const bool in = Rc[k] >= 0;  // a boundary edge reads its left cell twice
        const GpHead<R> *hl = head + rec_at(T, L[k], GKS_IX(sl[k] & 3, 3), g);
        const GpHead<R> *hr = in ? head + rec_at(T, Rc[k], GKS_IX(sl[k] >> 2, 3), 1 - g) : hl;
        z[k][0] = hl->h[hq];
        z[k][1] = hr->h[hq];
#pragma unroll
        for (int i = 0; i < 2; i++) {
            q[k][i] = hl->q[mq + i];
            q[k][2 + i] = hr->q[mq + i];
        }
        geo[k][0] = en[e[k]];
        geo[k][1] = en[E + e[k]];
        geo[k][2] = m.eBgp[g * E + e[k]];
        geo[k][3] = m.gg[(2 * k) * T + c];
        geo[k][4] = m.gg[(2 * k + 1) * T + c];
    }
#pragma unroll
    for (int k = 0; k < 3; k++) {
        settle(geo[k]);
        settle(z[k]);
        settle(q[k]);
    }
    double sx = 0, sy = 0;
#pragma unroll
    for (int k = 0; k < 3; k++) {
        const double nx = geo[k][0], ny = geo[k][1], Bg = geo[k][2];
        // a dry side (thickness at or below h_dry, or not positive) has no velocity
        const double zl = z[k][0];
        const double hl = f == 0 ? zl - Bg : zl;
        const double unl = (hl > p.h_dry && hl > 0) ? ((double)q[k][0] * nx + (double)q[k][1] * ny) / hl : 0.0;
        double zr, hr, unr;
        if (Rc[k] >= 0) {
            zr = z[k][1];
            hr = f == 0 ? zr - Bg : zr;
            unr = (hr > p.h_dry && hr > 0) ? ((double)q[k][2] * nx + (double)q[k][3] * ny) / hr : 0.0;
        } else {  // mirror state across a wall; the same state across a free boundary
            zr = zl;
            hr = hl;
            unr = Rc[k] == -1 ? -unl : unl;
        }
        // reading: xi is the kinetic fraction of particles moving from left to right (one half
        // when both sides are dry)
        const double lb = 2.0 / (p.G * (hl + hr));
        const double xi = (hl + hr > 0) ? kinetic_fraction<R>(sqrt(lb) * 0.5 * (unl + unr)) : 0.5;
        const double hh = xi * zl + (1 - xi) * zr;
        const double h = 0.5 * hh + 0.5 * __shfl_xor(hh, 1);
        sx += geo[k][3] * h;
        sy += geo[k][4] * h;
    }
    gP1[(2 * f + g) * T + c] = g == 0 ? sx : sy;
}

// --------------------------------------------------------------------------------------------
// gas-kinetic evolution at one Gauss point for one layer (Sec. 2.2, Eq. SWE-2nd-order)
//
// Local frame: u along the edge normal.  Micro-slopes are Maxwellian-consistent (reading):
// a = alpha |c|^2 + beta c_u + gamma c_v with alpha = lam dh/h, beta = 2 lam dU, gamma = 2 lam dV,
// c = (u - U, v - V); the force term is -2 lam Phi . c.  Moments of the polynomial
//   P = a_n u + a_t v - 2 lam Phi . c
// over a (half-)Maxwellian are closed forms in the u-moments M_k and the centred v-moments.

// For the lower layer the bottom slope gB enters twice: in dh = d(eta1) - gB and in the force
// -G gB.  The |c|^2 part of the slope and the force part that carry gB are taken out of the
// polynomial P and added as the closed-form moments of
//   T_B = (gB_n/h)(2 c_u - lam |c|^2 u) + (gB_t/h)(2 c_v - lam |c|^2 v)
// (bottom_moments), whose momentum moments are exactly zero at rest in any precision, instead of
// two large terms that cancel.  The side record therefore carries the slopes of h (for beta,
// gamma) and of eta1 (for alpha), and the acceleration without its bottom part.
template <typename R>
struct SideL {
    R h, U, V;                    // state
    R ih;                         // 1/h
    R hn, ht, mnn, mnt, mtn, mtt;  // d/dn, d/dt of h, h U_n, h U_t
    R en, et;                     // d/dn, d/dt of the level whose |c|^2 slope enters P (h, or eta1)
    R pn, pt;                     // acceleration (without the bottom part for the lower layer)
};

template <typename R>
struct Slope {
    R an, bn, gn, at, bt, gt;
};

// ih = 1/h of the Maxwellian the slopes belong to
template <typename R>
__host__ __device__ inline Slope<R> slope_of(const SideL<R> &s, R ih, R U, R V, R lam)
{
    Slope<R> r;
    r.an = lam * s.en * ih;
    r.bn = 2 * lam * (s.mnn - U * s.hn) * ih;
    r.gn = 2 * lam * (s.mtn - V * s.hn) * ih;
    r.at = lam * s.et * ih;
    r.bt = 2 * lam * (s.mnt - U * s.ht) * ih;
    r.gt = 2 * lam * (s.mtt - V * s.ht) * ih;
    return r;
}

// out += <u^e psi T_B> for psi = (1, u, v) over a (half) Maxwellian with means (U, V), lam,
// th = 1/(2 lam) and u-moments M (the thickness cancels against the 1/h of T_B).  Closed forms
// from the moment recurrence M_{k+2} = U M_{k+1} + (k+1) th M_k and lam th = 1/2.
template <typename R>
__host__ __device__ inline void bottom_moments(R gn, R gt, R U, R V, R lam, R th, const R *M, int e, R *out)
{
    auto In = [&](int k) { return R(0.5 * (1 - k)) * M[k + 1] + R(0.5 * (k - 3)) * U * M[k]; };
    auto N1 = [&](int k) { return M[k + 1] - U * M[k]; };
    auto Jt = [&](int k) { return -V * (R(0.5 * (k + 2)) * M[k] - lam * U * N1(k)); };
    const R VV = V * V;
    auto Jv = [&](int k) {
        return M[k] * (R(0.5) * th - R(0.5) * VV - (VV + th) * R(0.5 * (k + 1))) + lam * U * (VV + th) * N1(k);
    };
    out[0] += gn * In(e) + gt * Jt(e);
    out[1] += gn * In(e + 1) + gt * Jt(e + 1);
    out[2] += gn * V * In(e) + gt * Jv(e);
}

// u-moments M_0..M_5 of the Gaussian (mean U, variance th = 1/(2 lam)) restricted to a half line
template <typename R>
__host__ __device__ inline void u_moments(R U, R th, R m0, R m1, R *M)
{
    M[0] = m0;
    M[1] = m1;
#pragma unroll
    for (int k = 2; k < 6; k++) M[k] = U * M[k - 1] + R(k - 1) * th * M[k - 2];
}

// moments of P (slope sl, force (pn, pt)) over a half Maxwellian with thickness h, means (U, V),
// lam, th = 1/(2 lam), u-moments M.  e = 0: <psi P>, e = 1: <u psi P>.
template <typename R>
__host__ __device__ inline void poly_moments(const Slope<R> &sl, R pn, R pt, R h, R U, R V, R lam, R th, const R *M, int e,
                                    R *out)
{
    R N1[5], N2[4];
#pragma unroll
    for (int k = 0; k < 5; k++) N1[k] = M[k + 1] - U * M[k];
#pragma unroll
    for (int k = 0; k < 4; k++) N2[k] = N1[k + 1] - U * N1[k];
    const R fn = sl.bt * V - 2 * lam * pn;
    const R q2 = sl.at * V + sl.gt;
    R Q[2];
#pragma unroll
    for (int i = 0; i < 2; i++) {
        const int j = e + i;
        Q[i] = sl.an * N2[j + 1] + sl.at * V * N2[j] + sl.bn * N1[j + 1] + fn * N1[j] +
               th * (sl.an * M[j + 1] + q2 * M[j]);
    }
    const R Rv = th * (sl.gn * M[e + 1] + (sl.gt * V - 2 * lam * pt) * M[e] + sl.at * N2[e] + sl.bt * N1[e]) +
                 3 * th * th * sl.at * M[e];
    out[0] = h * Q[0];
    out[1] = h * Q[1];
    out[2] = h * (V * Q[0] + Rv);
}

// a*b + c*d with both products rounded before the sum (no fused multiply-add): for mirror-image
// left/right contributions the result is then exactly zero, as a contracted fma(a, b, c*d) is not
template <typename R>
__host__ __device__ inline R sum_products(R a, R b, R c, R d)
{
#pragma clang fp contract(off)
    const R p = a * b, q = c * d;
    return p + q;
}

__host__ __device__ inline float erfc_(float x) { return erfcf(x); }
__host__ __device__ inline double erfc_(double x) { return erfc(x); }
__host__ __device__ inline float erf_(float x) { return erff(x); }
__host__ __device__ inline double erf_(double x) { return erf(x); }
__host__ __device__ inline float exp_(float x) { return expf(x); }
__host__ __device__ inline double exp_(double x) { return exp(x); }
__host__ __device__ inline float sqrt_(float x) { return sqrtf(x); }
__host__ __device__ inline double sqrt_(double x) { return sqrt(x); }

// Outputs (local frame): F0 with the hydrostatic term 1/2 G hb^2 removed from its normal-momentum
// component, Ft, Wb (hb_dev = hb - (hL + hR)/2 in slot 0), Wbt.  hbase = (hL + hR)/2 in FP64; the
// interface thickness is hbase + hb_dev.
// AM selects the constants alpha_{k,m} of the acceleration term (Sec. 2.2, Eq. SWE-2nd-order):
// AM = 0 the weights read for these slopes (below), AM = 1 the paper's printed (1, 3/4, 1/4) on the
// flux moments of the acceleration term in both the equilibrium and the initial distributions'
// parts, 1 on the state moments.
// Wet/dry (h_dry > 0): a vacuum side comes with h = 1/h = U = V = 0 and no slopes, so that each of
// its terms is an exact zero; an interface whose equilibrium thickness hbase + hdev is at or below
// h_dry gives zero outputs and returns true (dry).  order1: first order in time, F0 the step's mean
// flux F(dt)/dt and Ft = 0 (the caller passes sides without slopes and accelerations).
template <typename R, int AM = 0, int WD = 0>
__host__ __device__ inline bool gks_point(const SideL<R> &sl, const SideL<R> &sr, double hbase, R gBn, R gBt, R G, R eps,
                                 R eps_num, R dt, R *F0, R *Ft, R *Wb, R *Wbt, bool order1 = false,
                                 double h_dry = 0.0)
{
    // the bottom's moments are added unconditionally: for the upper layer (and a flat bottom) the
    // slope is zero and they add exact zeros.  A branch on the slope would diverge inside every wave,
    // whose lanes alternate between the layers in FP32
    // reciprocals formed once (lam = 1/(G h)); 1/(2 sqrt(pi lam)) = sqrt(lam) th / sqrt(pi)
    const R iG = div_(R(1), G), ihL = sl.ih, ihR = sr.ih;
    const R lamL = iG * ihL, lamR = iG * ihR;
    const R thL = R(0.5) * G * sl.h, thR = R(0.5) * G * sr.h;
    const R ispi = R(0.56418958354775628695);  // 1/sqrt(pi)
    R ML[6], MR[6], eL, eR;
    // half-space masses from one error function per Gaussian: 1/2 erfc(-x) = 1/2 (1 + erf(x))
    // (exactly 1/2 at rest; where erf(x) is close to -1 the lost relative digits of the tiny mass
    // are below the absolute rounding of the moments it enters)
    {
        const R sq = sqrt_(lamL);
        eL = erf_(sq * sl.U);  // 2 (M0 - 1/2)
        const R m0 = R(0.5) + R(0.5) * eL;
        const R ex = exp_(-lamL * sl.U * sl.U) * sq * thL * ispi;
        u_moments(sl.U, thL, m0, sl.U * m0 + ex, ML);
    }
    {
        const R sq = sqrt_(lamR);
        eR = -erf_(sq * sr.U);
        const R m0 = R(0.5) + R(0.5) * eR;  // 1/2 erfc(x)
        const R ex = exp_(-lamR * sr.U * sr.U) * sq * thR * ispi;
        u_moments(sr.U, thR, m0, sr.U * m0 - ex, MR);
    }
    // interface equilibrium state: thickness as an FP64 base plus a deviation that is 0 at rest
    const R hdev = R(0.5) * (sl.h * eL + sr.h * eR);
    if constexpr (WD) {
        if (!(hbase + (double)hdev > h_dry)) {  // no particles at the interface
#pragma unroll
            for (int i = 0; i < 3; i++) F0[i] = Ft[i] = Wb[i] = Wbt[i] = R(0);
            return true;
        }
    }
    const R hb = (R)(hbase + (double)hdev);
    const R wb1 = sum_products(sl.h, ML[1], sr.h, MR[1]);
    const R wb2 = sum_products(sl.h * ML[0], sl.V, sr.h * MR[0], sr.V);
    // brackets of the initial (side) distributions first, so that the sides' moments are dead
    // before the interface equilibrium's are formed.  B4 = (.., D4 + P + B4p, ..)
    R B4[3], B5[3], t1[3], t2[3];
    B4[0] = wb1;
    // normal momentum: h U M1 parts plus the pressure-like part's excess over 1/2 G hb^2
    // (h^2 M0 summed over the sides minus hb^2: exactly zero at rest)
    {
        const R sq2 = sum_products(sl.h * sl.h, ML[0], sr.h * sr.h, MR[0]);
        const R hb2 = sum_products(hb, hb, R(0), R(0));
        B4[1] = sum_products(sl.h * sl.U, ML[1], sr.h * sr.U, MR[1]) + R(0.5) * G * (sq2 - hb2);
    }
    B4[2] = sum_products(sl.h * ML[1], sl.V, sr.h * MR[1], sr.V);
    {
        const Slope<R> aL = slope_of(sl, ihL, sl.U, sl.V, lamL), aR = slope_of(sr, ihR, sr.U, sr.V, lamR);
        poly_moments(aL, sl.pn, sl.pt, sl.h, sl.U, sl.V, lamL, thL, ML, 1, t1);
        poly_moments(aR, sr.pn, sr.pt, sr.h, sr.U, sr.V, lamR, thR, MR, 1, t2);
        bottom_moments(gBn, gBt, sl.U, sl.V, lamL, thL, ML, 1, t1);
        bottom_moments(gBn, gBt, sr.U, sr.V, lamR, thR, MR, 1, t2);
#pragma unroll
        for (int i = 0; i < 3; i++) B5[i] = t1[i] + t2[i];
        if constexpr (AM == 1) {
            // the paper's constants on the initial distributions' acceleration moments: (3/4 - 1) on
            // <u u>, (1/4 - 1) on <u v>; the moments are -2 Phi_n N1_2 / G and
            // -2 (V Phi_n N1_1 + th Phi_t M_1) / G over each side's own half Maxwellian
            const R pLn = sl.pn - G * gBn, pLt = sl.pt - G * gBt, pRn = sr.pn - G * gBn, pRt = sr.pt - G * gBt;
            const R L1 = ML[2] - sl.U * ML[1], L2 = ML[3] - sl.U * ML[2];
            const R R1 = MR[2] - sr.U * MR[1], R2 = MR[3] - sr.U * MR[2];
            B5[1] += R(0.5) * iG * sum_products(pLn, L2, pRn, R2);
            B5[2] += R(1.5) * iG * (sl.V * pLn * L1 + thL * pLt * ML[1] + sr.V * pRn * R1 + thR * pRt * MR[1]);
        }
    }
    const R ihb = div_(R(1), hb);
    const R Ub = wb1 * ihb, Vb = wb2 * ihb;
    const R lamb = iG * ihb, thb = R(0.5) * G * hb;
    R Mp[6], Mm[6];
    {
        const R sq = sqrt_(lamb);
        const R eb = erf_(sq * Ub);
        const R m0p = R(0.5) + R(0.5) * eb, m0m = R(0.5) - R(0.5) * eb;
        const R ex = exp_(-lamb * Ub * Ub) * sq * thb * ispi;
        u_moments(Ub, thb, m0p, Ub * m0p + ex, Mp);
        u_moments(Ub, thb, m0m, Ub * m0m - ex, Mm);
    }
    const Slope<R> bL = slope_of(sl, ihb, Ub, Vb, lamb), bR = slope_of(sr, ihb, Ub, Vb, lamb);
    // time slope of the interface equilibrium from compatibility
    R wt[3];
    poly_moments(bL, sl.pn, sl.pt, hb, Ub, Vb, lamb, thb, Mp, 0, t1);
    poly_moments(bR, sr.pn, sr.pt, hb, Ub, Vb, lamb, thb, Mm, 0, t2);
    bottom_moments(gBn, gBt, Ub, Vb, lamb, thb, Mp, 0, t1);
    bottom_moments(gBn, gBt, Ub, Vb, lamb, thb, Mm, 0, t2);
    // well-balance weights of the acceleration in the equilibrium part (Sec. 2.2, the constants
    // alpha_{k,m} of Eq. SWE-2nd-order), read as the weights that make the half-space moments of a
    // balanced level slope and acceleration vanish for these slopes: 3/4 on <1>, 5/4 on <u u> and
    // <u v>, 1 elsewhere; applied relative to the full-space moments, so only the jump between the
    // sides' accelerations is weighted.  With h lam = 1/G the acceleration's moments are
    // -2 Phi_n N1_e / G (mass), -2 Phi_n N1_{e+1} / G, -2 (V Phi_n N1_e + th Phi_t M_e) / G.
    const R aLn = sl.pn - G * gBn, aLt = sl.pt - G * gBt, aRn = sr.pn - G * gBn, aRt = sr.pt - G * gBt;
    const R N1p0 = Mp[1] - Ub * Mp[0], N1m0 = Mm[1] - Ub * Mm[0];
    // mass, state moment: weight 3/4 (the full-space moment is zero); the paper's constants leave
    // the state moments unweighted
#pragma unroll
    for (int i = 0; i < 3; i++) wt[i] = -(t1[i] + t2[i]);
    if constexpr (AM == 0) wt[0] -= sum_products(aLn, N1p0, aRn, N1m0) * (R(0.5) * iG);
    // brackets multiplying the five time coefficients; B1 and B4 split into a hydrostatic part
    // and the rest.  B1 = (hb Ub, hb Ub^2 + P, hb Ub Vb)
    R B1[3], B2[3], B3[3];
    B1[0] = hb * Ub;
    B1[1] = hb * Ub * Ub;  // pressure removed
    B1[2] = hb * Ub * Vb;
    poly_moments(bL, sl.pn, sl.pt, hb, Ub, Vb, lamb, thb, Mp, 1, t1);
    poly_moments(bR, sr.pn, sr.pt, hb, Ub, Vb, lamb, thb, Mm, 1, t2);
    bottom_moments(gBn, gBt, Ub, Vb, lamb, thb, Mp, 1, t1);
    bottom_moments(gBn, gBt, Ub, Vb, lamb, thb, Mm, 1, t2);
#pragma unroll
    for (int i = 0; i < 3; i++) B2[i] = t1[i] + t2[i];
    {
        const R N1p1 = Mp[2] - Ub * Mp[1], N1m1 = Mm[2] - Ub * Mm[1];
        const R N1p2 = Mp[3] - Ub * Mp[2], N1m2 = Mm[3] - Ub * Mm[2];
        if constexpr (AM == 0) {
            // flux moments: weight 5/4 on the two momentum components; full-space parts from
            // N1_1 = th, N1_2 = 2 U th, M_1 = U
            const R sn = aLn + aRn, st = aLt + aRt, q = R(-0.5) * iG;  // (5/4 - 1) (-2 / G)
            B2[1] += q * (sum_products(aLn, N1p2, aRn, N1m2) - sn * Ub * thb);
            B2[2] += q * (Vb * sum_products(aLn, N1p1, aRn, N1m1) + thb * sum_products(aLt, Mp[1], aRt, Mm[1]) -
                          R(0.5) * thb * (sn * Vb + st * Ub));
        } else {
            // the paper's constants: (3/4 - 1) on <u u>, (1/4 - 1) on <u v> of the whole term
            B2[1] += R(0.5) * iG * sum_products(aLn, N1p2, aRn, N1m2);
            B2[2] += R(1.5) * iG * (Vb * sum_products(aLn, N1p1, aRn, N1m1) + thb * sum_products(aLt, Mp[1], aRt, Mm[1]));
        }
    }
    {
        const R aA = lamb * wt[0] * ihb;
        const R bA = 2 * lamb * (wt[1] - Ub * wt[0]) * ihb;
        const R gA = 2 * lamb * (wt[2] - Vb * wt[0]) * ihb;
        const R mA = 2 * aA * thb;  // <A>
        B3[0] = hb * (Ub * mA + bA * thb);
        B3[1] = hb * (Ub * Ub * mA + 2 * Ub * bA * thb + 4 * aA * thb * thb);
        B3[2] = hb * (Ub * Vb * mA + Ub * gA * thb + Vb * bA * thb);
    }
    // collision time (Sec. 4) in units of dt, and the weights of F(dt), F(dt/2) giving the flux and
    // its time derivative; c01 + c04 = 1 and ct1 + ct4 = 0 exactly (the hydrostatic part of B1 and B4
    // carries weight 1 in F0 and 0 in Ft)
    const R pl = sl.h * sl.h, pr = sr.h * sr.h;
    const R r = eps + eps_num * fabs(div_(pl - pr, pl + pr));
    const R E2 = exp_(div_(R(-0.5), r)), E1 = E2 * E2, a1 = 1 - E1, a2 = 1 - E2;
    // first order: the step's mean flux, c01 + c04 = 1 still, no time derivative
    const bool o1 = WD && order1;
    const R c04 = o1 ? r * a1 : r * (4 * a2 - a1), c01 = 1 - c04;
    const R ct1 = o1 ? R(0) : 4 * r * (2 * a2 - a1), ct4 = -ct1;
    const R c02 = -r + r * r * (8 * a2 - 2 * a1) - 2 * r * E2 + r * E1;
    const R ct2 = 4 * (2 * r * r * (a1 - 2 * a2) + r * (E2 - E1));
    const R c03 = -r + r * r * (4 * a2 - a1), ct3 = 4 * (R(0.25) + r * r * (a1 - 2 * a2));
    const R c05 = r * (2 + 4 * r) * E2 - r * (1 + r) * E1 - 3 * r * r;
    const R ct5 = 4 * (r * (1 + r) * E1 - r * (1 + 2 * r) * E2 + r * r);
    const R idt = div_(R(1), dt);
#pragma unroll
    for (int i = 0; i < 3; i++) {
        F0[i] = c01 * B1[i] + c04 * B4[i] + dt * (c02 * B2[i] + c03 * B3[i] + c05 * B5[i]);
        Ft[i] = (ct1 * B1[i] + ct4 * B4[i]) * idt + ct2 * B2[i] + ct3 * B3[i] + ct5 * B5[i];
    }
    Wb[0] = hdev;
    Wb[1] = wb1;
    Wb[2] = wb2;
    Wbt[0] = wt[0];
    Wbt[1] = wt[1];
    Wbt[2] = wt[2];
    return false;
}

// The same in FP64, with fewer operations: BOT = 0 leaves out the bottom's moments (the upper layer, whose
// bottom slope is zero), and at the interface
//   the half-space moments of the two sides' slopes about the one Maxwellian are taken as the full-space
//   moments of their mean (closed forms) plus the moments D = M(u > 0) - M(u < 0) of half their
//   difference: two sets of polynomial moments instead of four;
//   the bottom, the same on both sides, is left with its full-space moments -S (1, U, V) and
//   -S (U, U^2 + 2 th, U V), S = gB . (U, V), instead of four sets of half-space ones;
//   the well-balance weights of the acceleration apply to the difference alone as it stands.
// FP32 keeps the form above: any other order of its operations moves the results by the amplified rounding
// of a few obtuse cells (Fit).
template <int AM, int WD, int BOT>
__device__ inline bool gks_point64(const SideL<double> &sl, const SideL<double> &sr, double hbase, double gBn, double gBt, double G, double eps,
                                 double eps_num, double dt, double *F0, double *Ft, double *Wb, double *Wbt, bool order1,
                                 double h_dry)
{
    typedef double R;
    // reciprocals formed once (lam = 1/(G h)); 1/(2 sqrt(pi lam)) = sqrt(lam) th / sqrt(pi)
    const R iG = div_(R(1), G), ihL = sl.ih, ihR = sr.ih;
    const R lamL = iG * ihL, lamR = iG * ihR;
    const R thL = R(0.5) * G * sl.h, thR = R(0.5) * G * sr.h;
    const R ispi = R(0.56418958354775628695);  // 1/sqrt(pi)
    R ML[6], MR[6], eL, eR;
    // half-space masses from one error function per Gaussian: 1/2 erfc(-x) = 1/2 (1 + erf(x))
    // (exactly 1/2 at rest; where erf(x) is close to -1 the lost relative digits of the tiny mass
    // are below the absolute rounding of the moments it enters)
    {
        const R sq = sqrt_(lamL);
        eL = erf_(sq * sl.U);  // 2 (M0 - 1/2)
        const R m0 = R(0.5) + R(0.5) * eL;
        const R ex = exp_(-lamL * sl.U * sl.U) * sq * thL * ispi;
        u_moments(sl.U, thL, m0, sl.U * m0 + ex, ML);
    }
    {
        const R sq = sqrt_(lamR);
        eR = -erf_(sq * sr.U);
        const R m0 = R(0.5) + R(0.5) * eR;  // 1/2 erfc(x)
        const R ex = exp_(-lamR * sr.U * sr.U) * sq * thR * ispi;
        u_moments(sr.U, thR, m0, sr.U * m0 - ex, MR);
    }
    // interface equilibrium state: thickness as an FP64 base plus a deviation that is 0 at rest
    const R hdev = R(0.5) * (sl.h * eL + sr.h * eR);
    if constexpr (WD) {
        if (!(hbase + (double)hdev > h_dry)) {  // no particles at the interface
#pragma unroll
            for (int i = 0; i < 3; i++) F0[i] = Ft[i] = Wb[i] = Wbt[i] = R(0);
            return true;
        }
    }
    const R hb = (R)(hbase + (double)hdev);
    const R wb1 = sum_products(sl.h, ML[1], sr.h, MR[1]);
    const R wb2 = sum_products(sl.h * ML[0], sl.V, sr.h * MR[0], sr.V);
    // brackets of the initial (side) distributions first, so that the sides' moments are dead
    // before the interface equilibrium's are formed.  B4 = (.., D4 + P + B4p, ..)
    R B4[3], B5[3], t1[3], t2[3];
    B4[0] = wb1;
    // normal momentum: h U M1 parts plus the pressure-like part's excess over 1/2 G hb^2
    // (h^2 M0 summed over the sides minus hb^2: exactly zero at rest)
    {
        const R sq2 = sum_products(sl.h * sl.h, ML[0], sr.h * sr.h, MR[0]);
        const R hb2 = sum_products(hb, hb, R(0), R(0));
        B4[1] = sum_products(sl.h * sl.U, ML[1], sr.h * sr.U, MR[1]) + R(0.5) * G * (sq2 - hb2);
    }
    B4[2] = sum_products(sl.h * ML[1], sl.V, sr.h * MR[1], sr.V);
    {
        const Slope<double> aL = slope_of(sl, ihL, sl.U, sl.V, lamL), aR = slope_of(sr, ihR, sr.U, sr.V, lamR);
        poly_moments(aL, sl.pn, sl.pt, sl.h, sl.U, sl.V, lamL, thL, ML, 1, t1);
        poly_moments(aR, sr.pn, sr.pt, sr.h, sr.U, sr.V, lamR, thR, MR, 1, t2);
        if constexpr (BOT) {
            bottom_moments(gBn, gBt, sl.U, sl.V, lamL, thL, ML, 1, t1);
            bottom_moments(gBn, gBt, sr.U, sr.V, lamR, thR, MR, 1, t2);
        }
        settle(t1);
        settle(t2);
#pragma unroll
        for (int i = 0; i < 3; i++) B5[i] = t1[i] + t2[i];
        if constexpr (AM == 1) {
            // the paper's constants on the initial distributions' acceleration moments: (3/4 - 1) on
            // <u u>, (1/4 - 1) on <u v>; the moments are -2 Phi_n N1_2 / G and
            // -2 (V Phi_n N1_1 + th Phi_t M_1) / G over each side's own half Maxwellian
            const R pLn = sl.pn - G * gBn, pLt = sl.pt - G * gBt, pRn = sr.pn - G * gBn, pRt = sr.pt - G * gBt;
            const R L1 = ML[2] - sl.U * ML[1], L2 = ML[3] - sl.U * ML[2];
            const R R1 = MR[2] - sr.U * MR[1], R2 = MR[3] - sr.U * MR[2];
            B5[1] += R(0.5) * iG * sum_products(pLn, L2, pRn, R2);
            B5[2] += R(1.5) * iG * (sl.V * pLn * L1 + thL * pLt * ML[1] + sr.V * pRn * R1 + thR * pRt * MR[1]);
        }
    }
    const R ihb = div_(R(1), hb);
    const R Ub = wb1 * ihb, Vb = wb2 * ihb;
    const R lamb = iG * ihb, thb = R(0.5) * G * hb;
    // brackets multiplying the five time coefficients; B1 and B4 split into a hydrostatic part
    // and the rest.  B1 = (hb Ub, hb Ub^2 + P, hb Ub Vb), the pressure removed
    R B1[3], B2[3], B3[3], wt[3];
    const R sq = sqrt_(lamb), eb = erf_(sq * Ub);
    const R ex = exp_(-lamb * Ub * Ub) * sq * thb * ispi;
    R D[6];
    u_moments(Ub, thb, eb, Ub * eb + 2 * ex, D);
    const Slope<double> bL = slope_of(sl, ihb, Ub, Vb, lamb), bR = slope_of(sr, ihb, Ub, Vb, lamb);
    const Slope<double> d = {R(0.5) * (bL.an - bR.an), R(0.5) * (bL.bn - bR.bn), R(0.5) * (bL.gn - bR.gn),
                        R(0.5) * (bL.at - bR.at), R(0.5) * (bL.bt - bR.bt), R(0.5) * (bL.gt - bR.gt)};
    const R an = bL.an - d.an, bn = bL.bn - d.bn, gn = bL.gn - d.gn, at = bL.at - d.at, bt = bL.bt - d.bt, gt = bL.gt - d.gt;
    const R dpn = R(0.5) * (sl.pn - sr.pn), dpt = R(0.5) * (sl.pt - sr.pt);
    const R pn = sl.pn - dpn, pt = sl.pt - dpt;
    const R fn = bt * Vb - 2 * lamb * pn, w = gt * Vb - 2 * lamb * pt, atV = at * Vb;
    const R UU = Ub * Ub, UUt = UU + thb, UU4 = 2 * UU + 4 * thb, at4 = 4 * thb * at;
    const R S = BOT ? gBn * Ub + gBt * Vb : R(0), hth = hb * thb;
    const R q0 = hth * (2 * (Ub * an + atV) + bn + gt);
    const R q1 = hth * (UU4 * an + Ub * (2 * (atV + bn) + gt) + fn);
    const R q2 = hth * (Ub * (UU4 + 8 * thb) * an + UU4 * atV + UUt * (3 * bn + gt) + 2 * Ub * fn);
    const R v0 = hth * (gn * Ub + w + at4), v1 = hth * (gn * UUt + Ub * (w + at4) + bt * thb);
    B1[0] = hb * Ub;
    B1[1] = hb * UU;
    B1[2] = hb * Ub * Vb;
    // time slope of the interface equilibrium from compatibility, and the bracket of the slopes
    poly_moments(d, dpn, dpt, hb, Ub, Vb, lamb, thb, D, 0, t1);
    poly_moments(d, dpn, dpt, hb, Ub, Vb, lamb, thb, D, 1, t2);
    wt[0] = S - (t1[0] + q0);
    wt[1] = S * Ub - (t1[1] + q1);
    wt[2] = S * Vb - (t1[2] + (Vb * q0 + v0));
    B2[0] = t2[0] + q1 - S * Ub;
    B2[1] = t2[1] + q2 - S * (UUt + thb);
    B2[2] = t2[2] + (Vb * q1 + v1) - S * Ub * Vb;
    // the well-balance weights of the acceleration
    const R D1 = D[2] - Ub * D[1], D2 = D[3] - Ub * D[2];
    if constexpr (AM == 0) {
        wt[0] -= iG * dpn * ex;
        const R q = R(-0.5) * iG;
        B2[1] += q * dpn * D2;
        B2[2] += q * (Vb * dpn * D1 + thb * dpt * D[1]);
    } else {
        const R gn2 = pn - G * gBn, gt2 = pt - G * gBt;
        B2[1] += R(0.5) * iG * (2 * Ub * thb * gn2 + dpn * D2);
        B2[2] += R(1.5) * iG * (Vb * (thb * gn2 + dpn * D1) + thb * (Ub * gt2 + dpt * D[1]));
    }
    {
        const R aA = lamb * wt[0] * ihb;
        const R bA = 2 * lamb * (wt[1] - Ub * wt[0]) * ihb;
        const R gA = 2 * lamb * (wt[2] - Vb * wt[0]) * ihb;
        const R mA = 2 * aA * thb;  // <A>
        B3[0] = hb * (Ub * mA + bA * thb);
        B3[1] = hb * (Ub * Ub * mA + 2 * Ub * bA * thb + 4 * aA * thb * thb);
        B3[2] = hb * (Ub * Vb * mA + Ub * gA * thb + Vb * bA * thb);
    }
    // collision time (Sec. 4) in units of dt, and the weights of F(dt), F(dt/2) giving the flux and
    // its time derivative; c01 + c04 = 1 and ct1 + ct4 = 0 exactly (the hydrostatic part of B1 and B4
    // carries weight 1 in F0 and 0 in Ft)
    const R pl = sl.h * sl.h, pr = sr.h * sr.h;
    const R r = eps + eps_num * fabs(div_(pl - pr, pl + pr));
    const R E2 = exp_(div_(R(-0.5), r)), E1 = E2 * E2, a1 = 1 - E1, a2 = 1 - E2;
    // first order: the step's mean flux, c01 + c04 = 1 still, no time derivative
    const bool o1 = WD && order1;
    const R c04 = o1 ? r * a1 : r * (4 * a2 - a1), c01 = 1 - c04;
    const R ct1 = o1 ? R(0) : 4 * r * (2 * a2 - a1), ct4 = -ct1;
    const R c02 = -r + r * r * (8 * a2 - 2 * a1) - 2 * r * E2 + r * E1;
    const R ct2 = 4 * (2 * r * r * (a1 - 2 * a2) + r * (E2 - E1));
    const R c03 = -r + r * r * (4 * a2 - a1), ct3 = 4 * (R(0.25) + r * r * (a1 - 2 * a2));
    const R c05 = r * (2 + 4 * r) * E2 - r * (1 + r) * E1 - 3 * r * r;
    const R ct5 = 4 * (r * (1 + r) * E1 - r * (1 + 2 * r) * E2 + r * r);
    const R idt = div_(R(1), dt);
#pragma unroll
    for (int i = 0; i < 3; i++) {
        F0[i] = c01 * B1[i] + c04 * B4[i] + dt * (c02 * B2[i] + c03 * B3[i] + c05 * B5[i]);
        Ft[i] = (ct1 * B1[i] + ct4 * B4[i]) * idt + ct2 * B2[i] + ct3 * B3[i] + ct5 * B5[i];
    }
    Wb[0] = hdev;
    Wb[1] = wb1;
    Wb[2] = wb2;
    Wbt[0] = wt[0];
    Wbt[1] = wt[1];
    Wbt[2] = wt[2];
    return false;
}

// Time derivative of one side's own state (h, m.n, m.t in the local frame) from the shallow-water
// equations on that side's data: minus the derivative of the normal and tangential fluxes plus
// h times the acceleration; the pressure term takes the slope of the level (eta1 for the lower
// layer, whose bottom slope it contains, h2 for the upper).
template <typename R>
__device__ inline void side_rate(const SideL<R> &q, R G, R *o)
{
    const R U = q.U, V = q.V, h = q.h;
    o[0] = -(q.mnn + q.mtt);
    o[1] = -(R(2) * U * q.mnn - U * U * q.hn + G * h * q.en) - (U * q.mtt + V * q.mnt - U * V * q.ht) + h * q.pn;
    o[2] = -(U * q.mtn + V * q.mnn - U * V * q.hn) - (R(2) * V * q.mtt - V * V * q.ht + G * h * q.et) + h * q.pt;
}

// whether a wave of k_flux holds 32 edges of one layer (FP64: the layers take different paths through
// gks_point64) or 16 edges of both
template <typename R>
constexpr bool LAYER_WAVES = sizeof(R) == 8;

// one thread per (edge, Gauss point, layer); the two Gauss points of an edge are adjacent lanes
//
// Bound by latency and by the rate of issue: three waves a SIMD (152 registers in FP64), half of the
// time with no instruction ready, at 690 MB a launch on 520k cells in FP64 (132 us at the rate of a
// large copy).  The two stages on average, FP64: 520k cells 191 us with gks_point and both layers in
// a wave, 174 so; 800 cells 7.8, 6.5.  At 128 registers for four waves it spills (209).
// STAGE 1 (the second stage) writes only what the second update reads: the mass fluxes, the time
// derivatives, the interface thicknesses and the coupling's Gauss-point thicknesses and rates; the
// momentum fluxes, the hydrostatic terms and the interface momenta keep the first stage's values.
// GM = 1: the discontinuous reading of the gradient update: besides the fluxes, each side's own
// state and time derivative, averaged over the edge's two Gauss points (left side in the rows of
// the interface state, right side in eoh rows 6-7 and eom rows 24-33)
// WD = 1: wet/dry layers (Phys::h_dry > 0): vacuum sides, first-order band edges, dry interfaces;
// a template argument so that the wet-only path carries none of it
template <typename R, int AM, int STAGE, int GM, int WD, int LAY>
__device__ inline void flux_at(const MeshDev &m, const Phys &p, const GpRecs<R> &rec, const R *__restrict__ r0,
                               const double *__restrict__ gP1, double *__restrict__ eoh, R *__restrict__ eom, int64_t idx)
{
    const int g = idx & 1, lay = LAY;
    const int64_t e = (idx >> 7) * 32 + ((idx & 63) >> 1);
#include "gks_flux_body.h"
}

template <typename R, int AM, int STAGE, int GM = 0, int WD = 0>
__global__ void __launch_bounds__(256) k_flux(MeshDev m, Phys p, GpRecs<R> rec,
                                              const R *__restrict__ r0, const double *__restrict__ gP1,
                                              double *__restrict__ eoh, R *__restrict__ eom)
{
    const int64_t idx = xcd_block() * blockDim.x + threadIdx.x;
    if constexpr (LAYER_WAVES<R>) {
        if (__builtin_amdgcn_readfirstlane((int)(idx >> 6) & 1) == 0)
            flux_at<R, AM, STAGE, GM, WD, 0>(m, p, rec, r0, gP1, eoh, eom, idx);
        else
            flux_at<R, AM, STAGE, GM, WD, 1>(m, p, rec, r0, gP1, eoh, eom, idx);
    } else {
        constexpr int LAY = -1;
        const int64_t e = idx >> 2;
        const int g = idx & 1, lay = (idx >> 1) & 1;  // lay 0: lower layer (h1), 1: upper (h2)
#include "gks_flux_body.h"
    }
}

// --------------------------------------------------------------------------------------------
// cell update: deterministic gather of the three edges in FP64, sources, S2O4 stage update

// stage 0: Ws = W + dt/2 L + dt^2/8 Lt, gWs = G + dt/2 Gt; carry Wc = W + dt L + dt^2/6 Lt, Gc = G
// stage 1: W = Wc + dt^2/3 Lt, gW = Gc + dt Gt
// STAGE is a template argument: the second stage needs only the time derivatives, the thickness
// fluxes and the interface thicknesses, so it neither loads nor sums the momentum fluxes, the
// hydrostatic terms and the interface momenta
// SRC = 1: the higher-order layer coupling: the cell-average thickness in place of the Gauss-point
// mean, its rate from the cell's mass flux, plus the interior correction src[8][T] of k_recon.
// GM = 1: the discontinuous reading of the gradient update: a cell takes the interface values of
// its own side of each edge (the right cell of an edge reads eoh rows 6-7 and eom rows 24-33).
//
// Two lanes a cell, lane l layer l (0 upper, 1 lower), the other layer's slopes by a swap in the pair; a
// cell's lanes also write its ghosts in the new state, so that the next stage starts with the
// reconstruction, and in the second stage the wave speeds.  Bound by memory where the mesh is large: at
// 520k cells FP64 the first stage moves 441 MB, 85 us at the rate of a large copy, in 127 us, the second
// 331 MB, 64 us, in 82.
// By itself it is slower than one thread a cell was, whose two stages took 104.3 us on average, between
// events, where these take 108.7 without the wave speeds; the kernel for the ghosts, 8.9, is gone
// (180k FP32: 26.8, 25.1 + 6.7; 10k FP64: 9.1, 9.7 + 6.8).  With the ghosts written by one thread a cell
// it spills (134.9, 28.5, 14.4); the edges' values in blocks of 16 edges instead of rows change nothing
// (112.0, 73.0 at 520k FP32 / 72.9).
template <typename R, int STAGE, int SRC = 0, int GM = 0>
__global__ void __launch_bounds__(256) k_update(MeshDev m, Phys p, const double *__restrict__ eoh, const R *__restrict__ eom,
                                                const LayerW<R> *__restrict__ Win, const LayerG<R> *__restrict__ Gin,
                                                LayerW<R> *__restrict__ Wout, LayerG<R> *__restrict__ Gout,
                                                double *__restrict__ Wc, R *__restrict__ Gc, const R *__restrict__ src)
{
    const int64_t idx = xcd_block() * blockDim.x + threadIdx.x, c = idx >> 1;
    const int l = idx & 1;
    const bool lower = l == 1;
    if (c >= m.T) return;
    const int64_t T = m.T, E = m.E;
    const int sc = m.cscen ? (int)GKS_IX(m.cscen[c], m.S) : 0;
    const double dt = p.scal[2 * sc], G = p.G;
    LayerW<R> w;  // the stage's output
    LayerG<R> g;
    if (dt == 0.0) {
        // the scenario has reached its end time: the state stays as it is (the stage's output is
        // its input; stage 0 also leaves the carry equal to it for stage 1)
        if constexpr (STAGE == 0) {
            w = Win[idx];
            g = Gin[idx];
            Wc[idx] = w.h;
            Wc[2 * T + idx] = w.m[0];
            Wc[4 * T + idx] = w.m[1];
#pragma unroll
            for (int i = 0; i < 6; i++) Gc[2 * i * T + idx] = g.g[i];
        } else {
            w = {Wc[idx], {(R)Wc[2 * T + idx], (R)Wc[4 * T + idx]}};
#pragma unroll
            for (int i = 0; i < 6; i++) g.g[i] = Gc[2 * i * T + idx];
        }
    } else {
        // K: what couples the other layer's thickness into this one, G or chi G
        const double K = lower ? p.chi[sc] * G : G;
        double LF[3] = {0}, LFt[3] = {0}, GG[3][2] = {{0}}, GGt[3][2] = {{0}}, hs = 0, hts = 0;
        // smallest acceptable new thickness, exclusive: 0, or -h_dry with wet/dry layers
        const double hneg = p.h_dry > 0 ? -p.h_dry : 0.0;
        double GC[2] = {0, 0}, GCt[2] = {0, 0};  // central thickness
        const double *eh = eoh + l * E;
        const R *e1 = eom + (22 + l) * E, *e2 = eom + (12 + 2 * l) * E, *e3 = eom + 3 * l * E;
#pragma unroll
        for (int k = 0; k < 3; k++) {
            const int32_t code = m.cedge[k * T + c];
            const int64_t e = GKS_IX(code >= 0 ? code : ~code, m.E);
            const double f = m.fl[k * T + c], gx = m.gg[(2 * k) * T + c], gy = m.gg[(2 * k + 1) * T + c];
            // rows of this cell's interface values: shared, or those of its own side (GM = 1)
            const int64_t ho = (GM == 1 && code < 0) ? 4 * E : 0, mo = (GM == 1 && code < 0) ? 12 * E : 0;
            double Wb[3];
            Wb[0] = eh[2 * E + ho + e];
            if constexpr (STAGE == 0) {
                Wb[1] = e2[mo + e];
                Wb[2] = e2[E + mo + e];
            }
#pragma unroll
            for (int q = 0; q < 3; q++) {
                if (STAGE == 0 || q == 0) {
                    LF[q] -= f * (double)e3[q * E + e];
                    GG[q][0] += gx * Wb[q];
                    GG[q][1] += gy * Wb[q];
                }
                const double Ft = e3[(6 + q) * E + e];
                const double Wbt = e3[(16 + q) * E + mo + e];
                LFt[q] -= f * Ft;
                GGt[q][0] += gx * Wbt;
                GGt[q][1] += gy * Wbt;
            }
            if constexpr (STAGE == 0) {
                // hydrostatic part of the normal momentum flux, along the outward normal
                const double P = eh[e];
                LF[1] -= gx * P;
                LF[2] -= gy * P;
            }
            const double C = eh[4 * E + e], Ct = e1[e];
            GC[0] += gx * C;
            GC[1] += gy * C;
            GCt[0] += gx * Ct;
            GCt[1] += gy * Ct;
            hs += C;
            hts += Ct;
        }
        const double third = 1.0 / 3.0;
        hs *= third;
        hts *= third;
        // the other layer's slopes
#pragma unroll
        for (int d = 0; d < 2; d++) {
            GC[d] = __shfl_xor(GC[d], 1);
            GCt[d] = __shfl_xor(GCt[d], 1);
        }
        const double gBx = m.gB[c], gBy = m.gB[T + c];
        // rows of the interior correction: 0, 1 lower, 2, 3 upper, 4 .. 7 their rates
        const R *sr = SRC == 1 ? src + (lower ? 0 : 2) * T + c : nullptr;
        const double Bb = lower ? m.Bbar[c] : 0.0;
        LayerW<R> wi;
        double h = 0;
        if constexpr (STAGE == 0 || SRC == 1) {
            wi = Win[idx];
            h = wi.h - Bb;
        }
        // bottom source rate via the thickness rates; layer coupling rate by the product rule
        double Lt[3] = {LFt[0], LFt[1], LFt[2]};
        Lt[1] += LF[0] * (-G * gBx);
        Lt[2] += LF[0] * (-G * gBy);
        if constexpr (SRC == 1) {
            // higher order: cell-average thicknesses, their rates from the mass fluxes
            Lt[1] += -K * (LF[0] * GC[0] + h * GCt[0] + (double)sr[4 * T]);
            Lt[2] += -K * (LF[0] * GC[1] + h * GCt[1] + (double)sr[5 * T]);
        } else {
            Lt[1] += -K * (hts * GC[0] + hs * GCt[0]);
            Lt[2] += -K * (hts * GC[1] + hs * GCt[1]);
        }
        bool bad = false;  // a new thickness <= 0 (or NaN), or a non-finite momentum (via their sum)
        double msum = 0;
        if constexpr (STAGE == 0) {
            double L[3] = {LF[0], LF[1], LF[2]};
            // bottom source h_j (0, -G B_x, -G B_y) (Sec. 3.2) and layer coupling
            // (Eq. SWE-source-discretization) from the Gauss-point mean thickness and the Green-Gauss
            // derivative of the other layer's Gauss-point thickness (central values); the higher-order
            // form takes the cell average and adds the interior correction
            if constexpr (SRC == 1) {
                L[1] += h * (-G * gBx) - K * (h * GC[0] + (double)sr[0]);
                L[2] += h * (-G * gBy) - K * (h * GC[1] + (double)sr[T]);
            } else {
                L[1] += h * (-G * gBx) - K * hs * GC[0];
                L[2] += h * (-G * gBy) - K * hs * GC[1];
            }
            if (lower) {  // the state carries grad(eta1) = grad(h1) + grad(B)
                GG[0][0] += gBx;
                GG[0][1] += gBy;
            }
            const double bot = wi.h - h;  // the cell's bottom mean (lower layer)
#pragma unroll
            for (int q = 0; q < 3; q++) {
                const double wv = q == 0 ? wi.h : (double)wi.m[q == 2];
                const double ws = wv + 0.5 * dt * L[q] + 0.125 * dt * dt * Lt[q];
                if (q == 0)
                    w.h = ws;
                else
                    w.m[q == 2] = (R)ws;
                // a thickness <= 0 is bad, or with wet/dry layers one below -h_dry (a dry cell may hold
                // a rounding residue)
                if (q == 0) bad = !(ws - bot > hneg);
                else msum += ws;
                Wc[2 * q * T + idx] = wv + dt * L[q] + (dt * dt / 6.0) * Lt[q];
#pragma unroll
                for (int d = 0; d < 2; d++) {
                    g.g[2 * q + d] = (R)(GG[q][d] + 0.5 * dt * GGt[q][d]);
                    Gc[2 * (2 * q + d) * T + idx] = (R)GG[q][d];
                }
            }
        } else {
#pragma unroll
            for (int q = 0; q < 3; q++) {
                const double wn = Wc[2 * q * T + idx] + (dt * dt / 3.0) * Lt[q];
                if (q == 0)
                    w.h = wn;
                else
                    w.m[q == 2] = (R)wn;
                if (q == 0) bad = !(wn - Bb > hneg);
                else msum += wn;
#pragma unroll
                for (int d = 0; d < 2; d++)
                    g.g[2 * q + d] = (R)((double)Gc[2 * (2 * q + d) * T + idx] + dt * GGt[q][d]);
            }
        }
        if (bad || !isfinite(msum)) atomicMin(p.bad, (unsigned long long)c);
    }
    Wout[idx] = w;
    Gout[idx] = g;
    if constexpr (STAGE == 1) max_speed(p, idx >> 6, sc, wave_speed(p, lower ? w.h - m.Bbar[c] : w.h, w.m));
    if (m.NG > 0) {
        const int32_t j1 = m.gfirst[c + 1];
        for (int32_t j = m.gfirst[c]; j < j1; j++) mirror(m, GKS_IX(m.gof[GKS_IX(j, m.NG)], m.NG), l, w, g, Wout, Gout);
    }
}

// an explicit step of a single scenario, clipped like the CFL step so that t never passes t_end
__global__ void k_set_dt(Phys p, double dt)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        const double t = p.scal[1];
        double tn = t + dt;
        if (tn > p.t_end[0]) {
            dt = fmax(0.0, p.t_end[0] - t);
            tn = fmax(t, p.t_end[0]);
        }
        p.scal[0] = dt;
        p.scal[1] = tn;
    }
}

// per-layer mass of cells [c0, c1): fixed-order block sums (deterministic)
template <typename R>
__global__ void __launch_bounds__(256) k_mass_partial(MeshDev m, const LayerW<R> *__restrict__ W, int64_t c0,
                                                      int64_t c1, double *__restrict__ part)
{
    __shared__ double sh[2][256];
    double a = 0, b = 0;
    for (int64_t c = c0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < c1; c += (int64_t)gridDim.x * blockDim.x) {
        a += m.area[c] * W[2 * c].h;
        b += m.area[c] * (W[2 * c + 1].h - m.Bbar[c]);
    }
    sh[0][threadIdx.x] = a;
    sh[1][threadIdx.x] = b;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            sh[0][threadIdx.x] += sh[0][threadIdx.x + s];
            sh[1][threadIdx.x] += sh[1][threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = sh[0][0];
        part[2 * blockIdx.x + 1] = sh[1][0];
    }
}

// values [i0, i1) of the snapshot a caller reads: W [6][T] (h1 = eta1 - B), then gradW [6][2][T]
// (grad h1 = grad eta1 - grad B), in double: those before m0, W's, into outW, those from m0 on, gradW's,
// into outG.  One read and one write per value, coalesced; the host used to unpack and convert them
// component by component (31 ms on 520,200 cells in FP64, of which the transfer over PCIe is 1.4 ms).
template <typename R>
__global__ void __launch_bounds__(256) k_snapshot(MeshDev m, const LayerW<R> *__restrict__ W, const LayerG<R> *__restrict__ G,
                                                  int64_t i0, int64_t m0, int64_t i1, double *__restrict__ outW,
                                                  double *__restrict__ outG)
{
    const int64_t i = i0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= i1) return;
    const int64_t T = m.T, row = i / T, c = i - row * T;
    double x;
    if (row < 6) {
        const int l = row >= 3, q = (int)row - 3 * l;
        const LayerW<R> &w = W[2 * c + l];
        x = q == 0 ? (l ? w.h - m.Bbar[c] : w.h) : (double)w.m[q - 1];
    } else {
        const int l = row >= 12, q = (int)row - 6 - 6 * l;
        x = G[2 * c + l].g[q];
        if (l && q < 2) x -= m.gB[q * T + c];
    }
    if (i < m0) outW[i - i0] = x;
    else outG[i - m0] = x;
}

// The checkpoint's arrays between the device's layout and the checkpoint's component-major one: h2 and
// eta1 [2][TG] in double, the momenta [4][TG], the gradients [12][TG]; TO_STATE from `raw` into the state,
// else the other way.  raw holds the first 2 TG values as doubles and the rest as R, from byte 16 TG on.
template <typename R, bool TO_STATE>
__global__ void __launch_bounds__(256) k_checkpoint(MeshDev m, LayerW<R> *__restrict__ W, LayerG<R> *__restrict__ G,
                                                    void *__restrict__ raw)
{
    const int64_t TG = m.T + m.NG, i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 18 * TG) return;
    const int64_t row = i / TG, c = i - row * TG;
    double *h = static_cast<double *>(raw);
    R *q = reinterpret_cast<R *>(h + 2 * TG);
    if (row < 2) {
        double &x = W[2 * c + row].h;
        if constexpr (TO_STATE) x = h[i]; else h[i] = x;
    } else {
        const int64_t j = i - 2 * TG;
        R &x = row < 6 ? W[2 * c + (row - 2) / 2].m[row & 1] : G[2 * c + (row - 6) / 6].g[(row - 6) % 6];
        if constexpr (TO_STATE) x = q[j]; else q[j] = x;
    }
}

// Per-step diagnostics of a scenario's cells [c0, c1) (Sec. 3.2's well-balance property: a lake
// at rest keeps U = 0 and both levels flat): per block the largest speed |h U| / h of each layer
// (desingularised in thin layers when h_dry > 0, as in the time step) and the largest and smallest
// levels eta1 = h1 + B and eta2 = eta1 + h2, as six maxima (the minima negated); the host takes
// the maxima over the blocks.  Grid-stride over the cells.
template <typename R>
__global__ void __launch_bounds__(256) k_diag_partial(MeshDev m, const LayerW<R> *__restrict__ W, int64_t c0,
                                                      int64_t c1, double h_dry, double *__restrict__ part)
{
    __shared__ double sh[6][256];
    double v[6] = {0.0, 0.0, -HUGE_VAL, -HUGE_VAL, -HUGE_VAL, -HUGE_VAL};
    for (int64_t c = c0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < c1; c += (int64_t)gridDim.x * blockDim.x) {
        const LayerW<R> wu = W[2 * c], wl = W[2 * c + 1];
        const double h2 = wu.h, e1 = wl.h, h1 = e1 - m.Bbar[c];
        const double m2x = wu.m[0], m2y = wu.m[1], m1x = wl.m[0], m1y = wl.m[1];
        v[0] = fmax(v[0], wd_velocity(h2, sqrt(m2x * m2x + m2y * m2y), h_dry));
        v[1] = fmax(v[1], wd_velocity(h1, sqrt(m1x * m1x + m1y * m1y), h_dry));
        v[2] = fmax(v[2], e1);
        v[3] = fmax(v[3], -e1);
        v[4] = fmax(v[4], e1 + h2);
        v[5] = fmax(v[5], -(e1 + h2));
    }
#pragma unroll
    for (int k = 0; k < 6; k++) sh[k][threadIdx.x] = v[k];
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
#pragma unroll
            for (int k = 0; k < 6; k++) sh[k][threadIdx.x] = fmax(sh[k][threadIdx.x], sh[k][threadIdx.x + s]);
        }
        __syncthreads();
    }
    if (threadIdx.x < 6) part[6 * blockIdx.x + threadIdx.x] = sh[threadIdx.x][0];
}

}  // namespace gks
