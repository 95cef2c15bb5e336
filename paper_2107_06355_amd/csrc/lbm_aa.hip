// In-place streaming with the AA access pattern (LBM_VARIANT_AA): one population buffer
// instead of two.
//
// Storage A_i[x] holds population i of node x.  Steps alternate between two access
// patterns, so that in every step each location is read and written by one node only:
//   even step t (natural layout): node x reads f_i(x, t) = A_i[x] and writes its
//     post-collision f*_i(x, t) to A_opp(i)[x] (its own node, opposite slot);
//   odd step t (swapped layout):  node x reads f_i(x, t) = f*_i(x - c_i, t - 1) =
//     A_opp(i)[x - c_i] and writes f*_i(x, t) to A_i[x + c_i], which is where the next
//     even step's node x + c_i reads f_i.
// Half-way bounce-back (walls) keeps that: in an odd step a population that would come from
// a solid node is f*_opp(i)(x, t - 1), which the even step left at A_i[x], and one that
// would go into a solid node is stored at A_opp(i)[x], where the even step's node x reads
// f_opp(i).  The rest population stays at its node.  After an even number of steps node x
// holds its own f_i(x, t) (the two-buffer variants hold the post-collision f*_i(x, t - 1)
// there and pull), after an odd number the swapped layout above.
//
// What the fused pull kernels cannot do here is form psi of the neighbours while updating
// a node (Eq. ShanChenForce): the densities of x + c_i live in locations those nodes
// overwrite during the same pass.  So each step is two launches: k_aa_psi writes psi of
// every node to a plane of the workspace, then k_aa_step reads psi of the 3 x 3 stencil
// from it, collides (node_collide, the same node arithmetic as every other variant) and
// writes in place.  Per FP32-shifted node update that is 80 B of populations plus 40 B
// read again and 8 B of psi: the variant halves the population memory, not the traffic.
#include "lbm_ctx.h"

namespace {

using namespace lbmk;

constexpr int kAaRows = 4;  // rows (one wavefront each) per 256-thread workgroup
constexpr int kOpp[9] = {0, 3, 4, 1, 2, 7, 8, 5, 6};

struct AaNode {
    int x, y;
    unsigned tile;  // 64 columns x kAaRows rows, row-major
    bool live;
};

// XCD-contiguous tiles (the grid is padded to a multiple of 8): the rows and lines that
// neighbouring tiles share, read by two kernels and nine stencils, are then found in one XCD's L2.
// Measured, us per step, tiles dealt out over the XCDs / contiguous: FP32 2048 x 1024 47.9 / 41.5,
// 8192^2 1799 / 1595, 1000^2 25.0 / 22.5; FP64 2048^2 191.8 / 188.1, 512^2 10.72 / 10.84.
__device__ __forceinline__ AaNode aa_node(const StepArgs& A)
{
    const unsigned cols = (unsigned)(A.nx + 63) / 64;
    AaNode n;
    n.tile = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const unsigned by = n.tile / cols;
    n.x = (int)(n.tile - by * cols) * 64 + (threadIdx.x & 63);
    n.y = (int)by * kAaRows + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    n.live = n.x < A.nx && n.y < A.ny;
    return n;
}

// Where a node and its neighbours lie: the rows (scalar, one row per wave) and columns with the
// periodic wrap, and whether the row below or above is a wall's.  A wave's loads then differ by
// row only in one branch, at the walls; tested neighbour by neighbour (nine to sixteen branches
// around single loads) FP64 2048^2 took 202.1 us per step
// against 191.8, FP32 8192^2 1812 against 1799.
struct AaPos {
    uint32_t r0, rm, rp;  // row offsets of y, y - 1, y + 1
    uint32_t x, xm, xp;
    bool bot, top;
};
__device__ __forceinline__ AaPos aa_pos(const StepArgs& A, int x, int y)
{
    const uint32_t ld = (uint32_t)A.ld;
    AaPos p;
    p.r0 = (uint32_t)y * ld;
    p.rm = (uint32_t)(y == 0 ? A.ny - 1 : y - 1) * ld;
    p.rp = (uint32_t)(y == A.ny - 1 ? 0 : y + 1) * ld;
    p.x = (uint32_t)x;
    p.xm = (uint32_t)(x == 0 ? A.nx - 1 : x - 1);
    p.xp = (uint32_t)(x == A.nx - 1 ? 0 : x + 1);
    p.bot = A.walls && y == 0;
    p.top = A.walls && y == A.ny - 1;
    return p;
}

// f_i(x, t) of the step with parity ODD, i = 0..8 (rest population in g0)
template <typename T, bool ODD>
__device__ __forceinline__ void aa_gather(const View<T>& V, const AaPos& p, double& g0, T g[9])
{
    const uint32_t own = p.r0 + p.x;
    g0 = ld_at<double>(V.rest, own);
    if (!ODD) {
#pragma unroll
        for (int i = 1; i < 9; ++i) g[i] = ld_at<T>(V.mv[i], own);
        return;
    }
    // from x - c_i; bounce-back from a solid node: the slot the even step left at x
    g[1] = ld_at<T>(V.mv[3], p.r0 + p.xm);
    g[3] = ld_at<T>(V.mv[1], p.r0 + p.xp);
    if (!p.bot) {
        g[2] = ld_at<T>(V.mv[4], p.rm + p.x);
        g[5] = ld_at<T>(V.mv[7], p.rm + p.xm);
        g[6] = ld_at<T>(V.mv[8], p.rm + p.xp);
    } else {
        g[2] = ld_at<T>(V.mv[2], own);
        g[5] = ld_at<T>(V.mv[5], own);
        g[6] = ld_at<T>(V.mv[6], own);
    }
    if (!p.top) {
        g[4] = ld_at<T>(V.mv[2], p.rp + p.x);
        g[7] = ld_at<T>(V.mv[5], p.rp + p.xp);
        g[8] = ld_at<T>(V.mv[6], p.rp + p.xm);
    } else {
        g[4] = ld_at<T>(V.mv[4], own);
        g[7] = ld_at<T>(V.mv[7], own);
        g[8] = ld_at<T>(V.mv[8], own);
    }
}

// store f*_i(x, t) of the step with parity ODD
template <typename T, bool ODD>
__device__ __forceinline__ void aa_scatter(const WView<T>& D, const AaPos& p, const T o[9], double o0)
{
    const uint32_t own = p.r0 + p.x;
    auto st = [&](int plane, uint32_t off, T v) { *(T*)(D.mv[plane] + off * (uint32_t)sizeof(T)) = v; };
    *(double*)(D.rest + own * 8u) = o0;
    if (!ODD) {
#pragma unroll
        for (int i = 1; i < 9; ++i) st(kOpp[i], own, o[i]);
        return;
    }
    // to x + c_i; into a wall: bounce back
    st(1, p.r0 + p.xp, o[1]);
    st(3, p.r0 + p.xm, o[3]);
    if (!p.top) {
        st(2, p.rp + p.x, o[2]);
        st(5, p.rp + p.xp, o[5]);
        st(6, p.rp + p.xm, o[6]);
    } else {
        st(4, own, o[2]);
        st(7, own, o[5]);
        st(8, own, o[6]);
    }
    if (!p.bot) {
        st(4, p.rm + p.x, o[4]);
        st(7, p.rm + p.xm, o[7]);
        st(8, p.rm + p.xp, o[8]);
    } else {
        st(2, own, o[4]);
        st(5, own, o[7]);
        st(6, own, o[8]);
    }
}

// Initial state in the natural layout: f_i(x, 0) = f^eq_i(rho0, u0) of the node itself (the
// two-buffer variants store the same populations one node upstream, for their first pull).
// In FP32-shifted storage the FP64 rest population takes what the node's eight FP32-rounded
// moving populations leave of rho0, as there.
template <typename T>
__global__ __launch_bounds__(256) void k_aa_init(StepArgs A, const double* rho0, const double* ux0, const double* uy0)
{
    const AaNode n = aa_node(A);
    if (!n.live) return;
    const size_t c = (size_t)n.y * A.nx + n.x, off = (size_t)n.y * A.ld + n.x;
    const double r = rho0[c], u = ux0 ? ux0[c] : 0.0, v = uy0 ? uy0[c] : 0.0;
    Plane<T>::restw(A.dst, A.plane)[off] = init_population<T>(0, r, u, v, A.rho_ref);
    for (int i = 1; i < 9; ++i) Plane<T>::movw(A.dst, A.plane, i)[off] = (T)init_population<T>(i, r, u, v, A.rho_ref);
}

// psi of the density the populations hold before a step of parity ODD, into plane psi
template <typename T, bool ODD>
__global__ __launch_bounds__(256) void k_aa_psi(StepArgs A, T* psi, int check)
{
    const AaNode n = aa_node(A);
    if (!n.live) return;
    const View<T> V = make_view<T>(A.src, A.plane);
    double g0;
    T g[9];
    aa_gather<T, ODD>(V, aa_pos(A, n.x, n.y), g0, g);
    psi[(size_t)n.y * A.ld + n.x] = node_psi<T>(A, node_drho<T>(g0, g), check != 0);
}

// One step of parity ODD in place: gather, Eq. ShanChenForce from the psi plane,
// node_collide, scatter.  MODE_STEP_REDUCE leaves one FP64 (mass, j_x, j_y) triple per
// workgroup in A.partials (blocks in row-major grid order); MODE_MACROS writes the
// macroscopic fields and stores nothing.
template <typename T, bool ODD, int MODE>
__global__ __launch_bounds__(256) void k_aa_step(StepArgs A, const T* psi)
{
    const AaNode n = aa_node(A);
    Acc acc = {0.0, 0.0, 0.0};
    if (n.live) {
        const View<T> V = make_view<T>(A.src, A.plane);
        Row<T> R;
        const AaPos p = aa_pos(A, n.x, n.y);
        aa_gather<T, ODD>(V, p, R.g0, R.g);
        const double dr = node_drho<T>(R.g0, R.g);
        // psi of the neighbours: beyond a wall the ghost psi of Eq. ShanChenForce, whatever was loaded
        auto at = [&](uint32_t row, uint32_t col) { return ld_at<T>((const char*)psi, row + col); };
        const T pc = at(p.r0, p.x), pw = at(p.r0, p.xm), pe = at(p.r0, p.xp);
        const T sw = at(p.rm, p.xm), so = at(p.rm, p.x), se = at(p.rm, p.xp);
        const T nw = at(p.rp, p.xm), no = at(p.rp, p.x), ne = at(p.rp, p.xp);
        const T lo = (T)A.psi_lo, hi = (T)A.psi_hi;
        T Ftx, Fty;
        force_tilde<T>(A, p.bot ? lo : sw, p.bot ? lo : so, p.bot ? lo : se, pw, pe, p.top ? hi : nw, p.top ? hi : no,
                       p.top ? hi : ne, Ftx, Fty);
        Lane L;
        L.lane = threadIdx.x & 63;
        L.x = n.x;
        L.xm = L.xp = 0;
        L.valid = L.interior = true;
        T o[9];
        double o0;
        if (node_collide<T, MODE>(A, L, n.y, R, dr, pc, Ftx, Fty, acc, o, o0))
            aa_scatter<T, ODD>(make_wview<T>(A.dst, A.plane), p, o, o0);
    }
    if (MODE == MODE_STEP_REDUCE || MODE == MODE_MACROS) {
        // fixed-order sums: lanes by wave_total, then the four waves in order
        __shared__ double sm[kAaRows][3];
        const double m = wave_total(acc.m), jx = wave_total(acc.x), jy = wave_total(acc.y);
        const int w = threadIdx.x >> 6;
        if ((threadIdx.x & 63) == kTotalLane) {
            sm[w][0] = m;
            sm[w][1] = jx;
            sm[w][2] = jy;
        }
        __syncthreads();
        if (threadIdx.x < 3) {
            double s = 0.0;
            for (int k = 0; k < kAaRows; ++k) s += sm[k][threadIdx.x];
            if (n.y < A.ny) A.partials[3 * (size_t)n.tile + threadIdx.x] = s;
        }
    }
}

// FP64 populations f_i = g_i + w_i rho_ref at their nodes, from either layout
template <typename T, bool ODD>
__global__ __launch_bounds__(256) void k_aa_populations(StepArgs A, double* out)
{
    const AaNode n = aa_node(A);
    if (!n.live) return;
    const View<T> V = make_view<T>(A.src, A.plane);
    double g0;
    T g[9];
    aa_gather<T, ODD>(V, aa_pos(A, n.x, n.y), g0, g);
    const size_t np = (size_t)A.nx * A.ny, o = (size_t)n.y * A.nx + n.x;
    out[o] = g0 + kW[0] * A.rho_ref;
    for (int i = 1; i < 9; ++i) out[i * np + o] = (double)g[i] + kW[i] * A.rho_ref;
}

unsigned aa_tiles(const lbm_params& p)
{
    return (unsigned)(p.nx + 63) / 64 * ((unsigned)(p.ny + kAaRows - 1) / kAaRows);
}
dim3 aa_grid(const lbm_params& p) { return dim3((aa_tiles(p) + 7) / 8 * 8); }

template <typename T>
bool aa_launch(lbm_ctx* c, int mode, hipStream_t s, double* const* macros)
{
    StepArgs A = c->args;
    A.src = c->buf[0];
    A.dst = c->buf[0];
    A.step = c->step;
    if (macros) {
        A.o_rho = macros[0];
        A.o_ux = macros[1];
        A.o_uy = macros[2];
        A.o_psi = macros[3];
        A.o_p = macros[4];
        A.o_fx = macros[5];
        A.o_fy = macros[6];
    }
    T* psi = (T*)c->aa_psi;
    const dim3 g = aa_grid(c->P), b(256);
    const bool odd = c->step & 1;
    const int check = mode != MODE_MACROS;
    if (odd) hipLaunchKernelGGL((k_aa_psi<T, true>), g, b, 0, s, A, psi, check);
    else hipLaunchKernelGGL((k_aa_psi<T, false>), g, b, 0, s, A, psi, check);
    const T* cpsi = psi;
    if (mode == MODE_STEP) {
        if (odd) hipLaunchKernelGGL((k_aa_step<T, true, MODE_STEP>), g, b, 0, s, A, cpsi);
        else hipLaunchKernelGGL((k_aa_step<T, false, MODE_STEP>), g, b, 0, s, A, cpsi);
    } else if (mode == MODE_STEP_REDUCE) {
        if (odd) hipLaunchKernelGGL((k_aa_step<T, true, MODE_STEP_REDUCE>), g, b, 0, s, A, cpsi);
        else hipLaunchKernelGGL((k_aa_step<T, false, MODE_STEP_REDUCE>), g, b, 0, s, A, cpsi);
    } else {
        if (odd) hipLaunchKernelGGL((k_aa_step<T, true, MODE_MACROS>), g, b, 0, s, A, cpsi);
        else hipLaunchKernelGGL((k_aa_step<T, false, MODE_MACROS>), g, b, 0, s, A, cpsi);
    }
    return hip_ok(hipGetLastError(), "k_aa_step launch");
}

}  // namespace

namespace lbmk {

int aa_slots(const lbm_params& p)
{
    return (int)aa_tiles(p);
}

size_t aa_psi_bytes(const lbm_params& p, int ld)
{
    const size_t t = p.prec == LBM_FP32_SHIFTED ? sizeof(float) : sizeof(double);
    return ((size_t)ld * p.ny * t + 255) & ~(size_t)255;
}

bool aa_step(lbm_ctx* c, int mode, hipStream_t s)
{
    return c->P.prec == LBM_FP32_SHIFTED ? aa_launch<float>(c, mode, s, nullptr)
                                         : aa_launch<double>(c, mode, s, nullptr);
}

bool aa_macros(lbm_ctx* c, double* const out[7], hipStream_t s)
{
    return c->P.prec == LBM_FP32_SHIFTED ? aa_launch<float>(c, MODE_MACROS, s, out)
                                         : aa_launch<double>(c, MODE_MACROS, s, out);
}

bool aa_init(lbm_ctx* c, const double* rho0, const double* ux0, const double* uy0, hipStream_t s)
{
    StepArgs A = c->args;
    A.dst = c->buf[0];
    const dim3 g = aa_grid(c->P), b(256);
    if (c->P.prec == LBM_FP32_SHIFTED) hipLaunchKernelGGL(k_aa_init<float>, g, b, 0, s, A, rho0, ux0, uy0);
    else hipLaunchKernelGGL(k_aa_init<double>, g, b, 0, s, A, rho0, ux0, uy0);
    return hip_ok(hipGetLastError(), "k_aa_init launch");
}

bool aa_populations(lbm_ctx* c, double* f_out, hipStream_t s)
{
    StepArgs A = c->args;
    A.src = c->buf[0];
    const dim3 g = aa_grid(c->P), b(256);
    const bool odd = c->step & 1, f32 = c->P.prec == LBM_FP32_SHIFTED;
    if (f32 && odd) hipLaunchKernelGGL((k_aa_populations<float, true>), g, b, 0, s, A, f_out);
    else if (f32) hipLaunchKernelGGL((k_aa_populations<float, false>), g, b, 0, s, A, f_out);
    else if (odd) hipLaunchKernelGGL((k_aa_populations<double, true>), g, b, 0, s, A, f_out);
    else hipLaunchKernelGGL((k_aa_populations<double, false>), g, b, 0, s, A, f_out);
    return hip_ok(hipGetLastError(), "k_aa_populations launch");
}

}  // namespace lbmk
