// liblbm.so: the finite-difference reference solver of the paper's appendix
// ("Finite Difference Method"), FP64; periodic in x, in y periodic or with the
// wall layers of the appendix's grid study.
//
// State: rho, u, v on an nx x ny mesh of spacing h (LBM units, c = 1,
// c_s^2 = 1/3).  One time step is the MacCormack predictor-corrector
//   Q* = Q^n + dt R+(Q^n),   Q^{n+1} = (Q^n + Q* + dt R-(Q*)) / 2
// with R the right-hand sides of the mass equation and Eq. FDmomentum: first
// derivatives of the convective, pressure and viscous terms are one-sided
// (forward in R+, backward in R-), second derivatives and every derivative of
// psi in Eq. FDforce are central; viscosities from Eq. DynamicViscosity with
// tau_nu(rho) of Eq. RelaxationTime (Eq. FDviscosityDerivative).
// One launch per step: each workgroup evaluates the predictor on its tile grown
// by two nodes in LDS and then the corrector on the tile, writing the new state
// to the second state buffer (the two buffers swap roles every step).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <utility>

#include "lbm.h"
#include "lbm_device.h"
#include "lbm_internal.h"

struct lbm_fd_ctx {
    lbm_fd_params P;
    lbmk::DevEos eos;
    double psi_wall;
    size_t n;
    double *rho, *u, *v, *rs, *us, *vs;
    unsigned* err;
    long long step;
};

namespace {

using namespace lbmk;

struct FdArgs {
    int nx, ny, var_tau, walls;
    double psi_wall;      // psi_l of Eq. B2
    double h, two_inv_G;
    double dt_h;                    // dt / h
    double k_mu, k_B;               // dt / h^2 times mu / rho and mu_B / rho (constant tau_nu)
    double k_tau, k_dtau;           // dt / h^2 times c_s^2, and that times dtau_nu / drho
    double f_g, f_L, f_s;           // dt G / (2 h^3) times the coefficients of Eq. FDforce
    double tau_e, tau_v, tau_lo, tau_hi, dtau, rho_v_tau;
    DevEos eos;
    unsigned* err;
    long long step;
};

__device__ __forceinline__ void fd_flag(const FdArgs& A)
{
    if (atomicCAS(A.err, 0u, 1u) == 0u) A.err[1] = (unsigned)A.step;
}

// One MacCormack step per launch.  A workgroup owns a kTx x kTy output tile.
// LDS holds the state, p_EOS and psi on the tile grown by 4 (region R4; the
// predictor at the tile grown by 2 reaches two more nodes through the
// Laplacian of psi in Eq. FDforce), then the predicted state, p_EOS and psi
// on the tile grown by 2 (region R2).  Ghost rows beyond the walls are
// written into both regions by the wall rules, so every stencil reads LDS
// with the same offsets.  Traffic per node-step: the state read once (plus
// the four-node ring, mostly from L2) and written once, and 28 bytes per thread of spilled registers.
//
// What bounds it (counters): at 512^2, two workgroups per CU in one round, latency: of 9.6 us, VALU
// issue takes 3.7 and LDS reads (41 per right-hand side) 3.5, and the waves wait half of their
// time.  At 4096^2, 445 us, issue takes 53%, LDS 50%, and the traffic, 1.70 GB, runs at 77% of the copy
// rate; 0.47 GB of it are the spilled registers' writes.  Measured (MI355X, us/step), with 512 threads
// and two rounds of predictor nodes, divided differences and integer remainders -> now: 512^2 10.6 ->
// 9.5, 2048^2 114 -> 99, 700 x 500 with walls and tau(rho) 17.1 -> 15.4, 200^2 7.3 -> 6.0.  Two nodes per thread share 30
// of 82 LDS reads but take 168 registers (12 instead of 24 waves per CU): 2048^2 140.
constexpr int kTx = 32, kTy = 16;
constexpr int kAx = kTx + 8, kAy = kTy + 8;   // R4
constexpr int kBx = kTx + 4, kBy = kTy + 4;   // R2

// dt times the right-hand sides of the mass equation and Eq. FDmomentum at LDS node (a, b)
// of arrays with row pitch P: one-sided first derivatives (DIR), central second
// derivatives, and Eq. FDforce from psi with central differences.  The differences are left
// undivided and the powers of h and dt folded into the constants of FdArgs.
template <int DIR, int P>
__device__ __forceinline__ void fd_rhs(const FdArgs& A, const double* R, const double* U, const double* V,
                                       const double* Pe, const double* S, int a, int b, double& dr, double& du,
                                       double& dv)
{
    const int c = b * P + a;
    const double r = R[c], ux = U[c], uy = V[c];
    const double ue = U[c + 1], uw = U[c - 1], un = U[c + P], us = U[c - P];
    const double ve = V[c + 1], vw = V[c - 1], vn = V[c + P], vs = V[c - P];
    // one-sided first differences
    const double rx = DIR > 0 ? R[c + 1] - r : r - R[c - 1], ry = DIR > 0 ? R[c + P] - r : r - R[c - P];
    const double u_x = DIR > 0 ? ue - ux : ux - uw, u_y = DIR > 0 ? un - ux : ux - us;
    const double v_x = DIR > 0 ? ve - uy : uy - vw, v_y = DIR > 0 ? vn - uy : uy - vs;
    const double px = DIR > 0 ? Pe[c + 1] - Pe[c] : Pe[c] - Pe[c - 1];
    const double py = DIR > 0 ? Pe[c + P] - Pe[c] : Pe[c] - Pe[c - P];
    const double div = u_x + v_y, t = v_x + u_y;
    dr = -A.dt_h * (r * div + (ux * rx + uy * ry));
    // central second differences of the velocity
    const double u_xx = (ue + uw) - 2.0 * ux, u_yy = (un + us) - 2.0 * ux;
    const double v_xx = (ve + vw) - 2.0 * uy, v_yy = (vn + vs) - 2.0 * uy;
    const double u_xy = 0.25 * ((U[c + P + 1] - U[c - P + 1]) - (U[c + P - 1] - U[c - P - 1]));
    const double v_xy = 0.25 * ((V[c + P + 1] - V[c - P + 1]) - (V[c + P - 1] - V[c - P - 1]));
    // divergence of the viscous stress (Eq. FDstressTensor) with Eq. DynamicViscosity: with
    // mu = r k, mu_B = r k_B it is k (D + r E) + k_B (rx div + r F), D and E the terms of the
    // viscosity's gradient and of the velocity's second derivatives
    const double Dx = 2.0 * (rx * u_x) + ry * t, Dy = rx * t + 2.0 * (ry * v_y);
    const double Fx = u_xx + v_xy, Fy = u_xy + v_yy;
    const double Ex = Fx + (u_xx + u_yy), Ey = Fy + (v_xx + v_yy);
    const double Bx = rx * div, By = ry * div;
    double k = A.k_mu, kB = A.k_B, Sx = 0.0, Sy = 0.0;
    if (A.var_tau) {
        // Eq. RelaxationTime and Eq. FDviscosityDerivative (zero where tau is clamped)
        double tn = A.tau_v + A.dtau * (r - A.rho_v_tau), kd = r * A.k_dtau;
        if (tn <= A.tau_lo) { tn = A.tau_lo; kd = 0.0; }
        if (tn >= A.tau_hi) { tn = A.tau_hi; kd = 0.0; }
        k = A.k_tau * (tn - 0.5);
        kB = A.k_tau * (A.tau_e - tn);
        Sx = kd * (Dx - Bx);
        Sy = kd * (Dy - By);
    }
    Sx += k * (Dx + r * Ex) + kB * (Bx + r * Fx);
    Sy += k * (Dy + r * Ey) + kB * (By + r * Fy);
    // psi's reads stay behind the velocity's arithmetic: with all 41 in flight the kernel spills more
    // than 8 of the 80 registers of 24 waves per CU (512^2 9.7 us/step instead of 9.5)
    __builtin_amdgcn_sched_barrier(0);
    // Eq. FDforce, central differences of psi (the Laplacian at x+-1, y+-1 reaches two nodes out)
    const double s0 = S[c], sxp = S[c + 1], sxm = S[c - 1], syp = S[c + P], sym = S[c - P];
    const double spp = S[c + P + 1], spm = S[c - P + 1], smp = S[c + P - 1], smm = S[c - P - 1];
    const double sx = sxp - sxm, sy = syp - sym;
    const double sxx = (sxp + sxm) - 2.0 * s0, syy = (syp + sym) - 2.0 * s0;
    const double de = spp - smm, dw = spm - smp;  // the diagonals
    const double sxy = 0.25 * ((spp - spm) - (smp - smm));
    const double L = sxx + syy;
    const double Lx = (S[c + 2] - S[c - 2]) - 4.0 * sx + (de + dw);
    const double Ly = (S[c + 2 * P] - S[c - 2 * P]) - 4.0 * sy + (de - dw);
    const double gx = sx * sxx + sy * sxy, gy = sx * sxy + sy * syy;
    const double Px = A.f_g * gx + (A.f_L * (sx * L) + A.f_s * (s0 * Lx));
    const double Py = A.f_g * gy + (A.f_L * (sy * L) + A.f_s * (s0 * Ly));
    // Eq. FDmomentum
    const double inv_r = fast_rcp(r);
    du = (Sx - A.dt_h * px - Px) * inv_r - A.dt_h * (ux * u_x + uy * u_y);
    dv = (Sy - A.dt_h * py - Py) * inv_r - A.dt_h * (ux * v_x + uy * v_y);
}

// Ghost rows of a region (pitch P, rows b with global row gj = j_base + b) from its
// fluid rows: b1 (gj = -1): rho and psi extrapolated, u = v = 0, p = p_EOS(rho_b1);
// b2 (gj = -2): psi of Eq. B2 only; above row ny-1: the mirror of rows ny-2, ny-3
// with u, v reversed.  Periodic lattices have no ghost rows.
template <int P, int NY>
__device__ __forceinline__ void fd_ghost_rows(const FdArgs& A, double* R, double* U, double* V, double* Pe,
                                              double* S, int j_base, int tid, int nthreads)
{
    for (int q = tid; q < P * NY; q += nthreads) {
        const int a = q % P, b = q / P, gj = j_base + b;
        const int c = b * P + a;
        if (gj == -1 || gj == -2) {
            const int c0 = (0 - j_base) * P + a, c1 = c0 + P;  // rows 0 and 1 (inside the region)
            const double b1 = 2.0 * S[c0] - S[c1];
            if (gj == -1) {
                R[c] = 2.0 * R[c0] - R[c1];
                U[c] = 0.0;
                V[c] = 0.0;
                Pe[c] = dev_eos_p(A.eos, R[c]);
                S[c] = b1;
            } else {
                S[c] = b1 + 2.0 * A.h * (A.psi_wall - b1);
            }
        } else if (gj >= A.ny && gj <= A.ny + 1) {
            const int cm = (2 * (A.ny - 1) - gj - j_base) * P + a;
            R[c] = R[cm];
            U[c] = -U[cm];
            V[c] = -V[cm];
            Pe[c] = Pe[cm];
            S[c] = S[cm];
        }
    }
}

// i mod n for i in [-4, n + SPAN): one compare each way on meshes at least SPAN wide (an integer
// remainder takes about 25 instructions)
template <int SPAN>
__device__ __forceinline__ int fd_wrap(int i, int n)
{
    if (n < SPAN) {
        i %= n;
        return i < 0 ? i + n : i;
    }
    return i < 0 ? i + n : (i >= n ? i - n : i);
}

// kFdThreads: the predictor's 720 nodes on R2 in one round of threads; the fill of R4 takes
// two, whose loads are all issued before the first is used
constexpr int kFdThreads = 768;
static_assert(kBx * kBy <= kFdThreads && kTx * kTy <= kFdThreads, "one node per thread");

// BASE, SHAPED (shape is not LBM_SHAPE_NONE): the EOS branches a launch cannot take are left out,
// with the constants that would hold scalar registers (41 spilled) for all three phases.
template <int BASE, bool SHAPED, bool NT>
__global__ __launch_bounds__(kFdThreads) __attribute__((amdgpu_waves_per_eu(6)))
void k_fd_step(FdArgs args, const double* rho, const double* u, const double* v, double* o_r, double* o_u, double* o_v)
{
    __shared__ double aR[kAy * kAx], aU[kAy * kAx], aV[kAy * kAx], aP[kAy * kAx], aS[kAy * kAx];
    __shared__ double bR[kBy * kBx], bU[kBy * kBx], bV[kBy * kBx], bP[kBy * kBx], bS[kBy * kBx];
    FdArgs A = args;
    A.eos.base = BASE;
    if (!SHAPED) A.eos.shape = LBM_SHAPE_NONE;
    constexpr int kFill = (kAx * kAy + kFdThreads - 1) / kFdThreads;
    const int tid = threadIdx.x;
    const int i0 = blockIdx.x * kTx, j0 = blockIdx.y * kTy;
    // 1. the state, p_EOS and psi on R4; the rows beyond the walls are filled afterwards
    double fr[kFill], fu[kFill], fv[kFill];
    bool have[kFill];
#pragma unroll
    for (int k = 0; k < kFill; ++k) {
        const int q = tid + k * kFdThreads, a = q % kAx, b = q / kAx;
        int gi = i0 - 4 + a, gj = j0 - 4 + b;
        have[k] = q < kAx * kAy && !(A.walls && (gj < 0 || gj >= A.ny));
        fr[k] = 1.0;
        fu[k] = fv[k] = 0.0;
        if (have[k]) {
            gi = fd_wrap<kAx>(gi, A.nx);
            gj = fd_wrap<kAy>(gj, A.ny);
            const size_t g = (size_t)gj * A.nx + gi;
            fr[k] = rho[g];
            fu[k] = u[g];
            fv[k] = v[g];
        }
    }
#pragma unroll
    for (int k = 0; k < kFill; ++k) {
        const int q = tid + k * kFdThreads;
        if (!have[k]) continue;
        const double r = fr[k], pe = dev_eos_p(A.eos, r);
        const double qq = (pe - r * (1.0 / 3.0)) * A.two_inv_G;
        if (!(r > 0.0) || !(qq >= 0.0)) fd_flag(A);
        aR[q] = r;
        aU[q] = fu[k];
        aV[q] = fv[k];
        aP[q] = pe;
        aS[q] = qq > 0.0 ? fast_sqrt_pos(qq) : 0.0;
    }
    __syncthreads();
    if (A.walls) {
        fd_ghost_rows<kAx, kAy>(A, aR, aU, aV, aP, aS, j0 - 4, tid, kFdThreads);
        __syncthreads();
    }
    // 2. predictor Q* = Q + dt R+(Q) on the fluid nodes of R2
    const int b2 = tid / kBx, gj2 = j0 - 2 + b2;
    if (tid < kBx * kBy && !(A.walls && (gj2 < 0 || gj2 >= A.ny))) {
        const int a = tid - b2 * kBx;
        double dr, du, dv;
        fd_rhs<+1, kAx>(A, aR, aU, aV, aP, aS, a + 2, b2 + 2, dr, du, dv);
        const int c = (b2 + 2) * kAx + a + 2;
        const double nr = aR[c] + dr;
        bR[tid] = nr;
        bU[tid] = aU[c] + du;
        bV[tid] = aV[c] + dv;
        const double pe = dev_eos_p(A.eos, nr);
        const double qq = (pe - nr * (1.0 / 3.0)) * A.two_inv_G;
        bP[tid] = pe;
        bS[tid] = qq > 0.0 ? fast_sqrt_pos(qq) : 0.0;
    }
    __syncthreads();
    if (A.walls) {
        fd_ghost_rows<kBx, kBy>(A, bR, bU, bV, bP, bS, j0 - 2, tid, kFdThreads);
        __syncthreads();
    }
    // 3. corrector Q^{n+1} = (Q + Q* + dt R-(Q*)) / 2 on the tile
    const int tx = tid % kTx, ty = tid / kTx;
    const int i = i0 + tx, j = j0 + ty;
    if (ty >= kTy || i >= A.nx || j >= A.ny) return;
    double dr, du, dv;
    fd_rhs<-1, kBx>(A, bR, bU, bV, bP, bS, tx + 2, ty + 2, dr, du, dv);
    const int cb = (ty + 2) * kBx + tx + 2, ca = (ty + 4) * kAx + tx + 4;
    const size_t g = (size_t)j * A.nx + i;
    const double nr = 0.5 * (aR[ca] + (bR[cb] + dr));
    const double nu = 0.5 * (aU[ca] + (bU[cb] + du));
    const double nv = 0.5 * (aV[ca] + (bV[cb] + dv));
    if constexpr (NT) {
        // streaming stores when both state buffers fit in the MALL (as the LBM kernels do)
        __builtin_nontemporal_store(nr, o_r + g);
        __builtin_nontemporal_store(nu, o_u + g);
        __builtin_nontemporal_store(nv, o_v + g);
    } else {
        o_r[g] = nr;
        o_u[g] = nu;
        o_v[g] = nv;
    }
}

FdArgs fd_args(const lbm_fd_ctx* c)
{
    const lbm_fd_params& P = c->P;
    FdArgs A;
    std::memset(&A, 0, sizeof(A));
    A.nx = P.nx;
    A.ny = P.ny;
    A.var_tau = P.var_tau;
    A.walls = P.walls;
    A.psi_wall = c->psi_wall;
    A.h = P.h;
    A.two_inv_G = 2.0 / P.G;
    A.dt_h = P.dt / P.h;
    A.k_tau = P.dt / (P.h * P.h) / 3.0;
    A.k_mu = A.k_tau * (P.tau_nu - 0.5);
    A.k_B = A.k_tau * (P.tau_e - P.tau_nu);
    const double f = 0.5 * P.dt * P.G / (P.h * P.h * P.h);
    A.f_g = f * (1.0 / 6.0 - 0.25 * P.eps);
    A.f_L = f / 12.0;
    A.f_s = f * 0.25;
    A.tau_e = P.tau_e;
    A.tau_v = P.tau_v;
    A.tau_lo = P.tau_l < P.tau_v ? P.tau_l : P.tau_v;
    A.tau_hi = P.tau_l < P.tau_v ? P.tau_v : P.tau_l;
    A.dtau = P.var_tau ? (P.tau_l - P.tau_v) / (P.rho_l_tau - P.rho_v_tau) : 0.0;
    A.k_dtau = A.k_tau * A.dtau;
    A.rho_v_tau = P.rho_v_tau;
    A.eos = c->eos;
    A.err = c->err;
    A.step = c->step;
    return A;
}

bool ok(hipError_t e, const char* what)
{
    if (e == hipSuccess) return true;
    char buf[256];
    std::snprintf(buf, sizeof(buf), "%s: %s", what, hipGetErrorString(e));
    lbm_set_error(buf);
    return false;
}

template <bool NT>
void fd_launch(bool pr, bool shaped, dim3 grd, hipStream_t s, const FdArgs& A, const lbm_fd_ctx* c)
{
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grd, dim3(kFdThreads), 0, s, A, (const double*)c->rho, (const double*)c->u,
                           (const double*)c->v, c->rs, c->us, c->vs);
    };
    if (pr && shaped) go(k_fd_step<LBM_BASE_PR, true, NT>);
    else if (pr) go(k_fd_step<LBM_BASE_PR, false, NT>);
    else if (shaped) go(k_fd_step<LBM_BASE_CS, true, NT>);
    else go(k_fd_step<LBM_BASE_CS, false, NT>);
}

constexpr size_t kFdArrays = 6;

}  // namespace

extern "C" {

int lbm_fd_layout(const lbm_fd_params* p, size_t* bytes)
{
    if (!p || p->nx < 3 || p->ny < 3 || !(p->h > 0) || !(p->dt > 0) || !(p->G < 0)) {
        lbm_set_error("lbm_fd_layout: need nx, ny >= 3, h > 0, dt > 0 and G < 0");
        return LBM_EINVAL;
    }
    if (bytes) *bytes = 256 + kFdArrays * (((size_t)p->nx * p->ny * sizeof(double) + 255) & ~(size_t)255);
    return LBM_OK;
}

int lbm_fd_init(lbm_fd_ctx** out, const lbm_fd_params* p, void* buf, size_t buf_bytes, const double* rho0,
                const double* u0, const double* v0, void* stream)
{
    size_t need = 0;
    if (!out || !buf || !rho0) return LBM_EINVAL;
    const int st = lbm_fd_layout(p, &need);
    if (st != LBM_OK) return st;
    if (buf_bytes < need) {
        lbm_set_error("lbm_fd_init: buffer smaller than lbm_fd_layout requires");
        return LBM_EINVAL;
    }
    if (p->var_tau && !(p->rho_l_tau > p->rho_v_tau)) {
        lbm_set_error("lbm_fd_init: Eq. RelaxationTime needs rho_l_tau > rho_v_tau");
        return LBM_EINVAL;
    }
    lbm_fd_ctx* c = new (std::nothrow) lbm_fd_ctx();
    if (!c) return LBM_EINVAL;
    c->P = *p;
    c->eos = dev_eos(p->eos);
    {
        const double q = 2.0 * (lbm_eos_pressure(&p->eos, p->eos.rho_l) - p->eos.rho_l / 3.0) / p->G;
        c->psi_wall = q > 0.0 ? std::sqrt(q) : 0.0;  // psi_l of Eq. B2
    }
    c->n = (size_t)p->nx * p->ny;
    char* b = (char*)buf;
    c->err = (unsigned*)b;
    b += 256;
    const size_t arr = (c->n * sizeof(double) + 255) & ~(size_t)255;
    double** slots[kFdArrays] = {&c->rho, &c->u, &c->v, &c->rs, &c->us, &c->vs};
    for (size_t k = 0; k < kFdArrays; ++k, b += arr) *slots[k] = (double*)b;
    hipStream_t s = (hipStream_t)stream;
    const size_t nb = c->n * sizeof(double);
    bool good = ok(hipMemsetAsync(c->err, 0, 256, s), "fd clear") &&
                ok(hipMemcpyAsync(c->rho, rho0, nb, hipMemcpyDeviceToDevice, s), "fd rho0");
    good = good && (u0 ? ok(hipMemcpyAsync(c->u, u0, nb, hipMemcpyDeviceToDevice, s), "fd u0")
                       : ok(hipMemsetAsync(c->u, 0, nb, s), "fd u0"));
    good = good && (v0 ? ok(hipMemcpyAsync(c->v, v0, nb, hipMemcpyDeviceToDevice, s), "fd v0")
                       : ok(hipMemsetAsync(c->v, 0, nb, s), "fd v0"));
    if (!good) {
        delete c;
        return LBM_EHIP;
    }
    *out = c;
    return LBM_OK;
}

int lbm_fd_step(lbm_fd_ctx* c, int64_t nsteps, void* stream)
{
    if (!c || nsteps < 0) return LBM_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    const dim3 grd((c->P.nx + kTx - 1) / kTx, (c->P.ny + kTy - 1) / kTy);
    // streaming stores when both state buffers (2 x 3 fields x 8 B per node) are small
    const bool nt = (size_t)c->P.nx * c->P.ny * 48 <= kStreamBytes;
    for (int64_t t = 0; t < nsteps; ++t) {
        FdArgs A = fd_args(c);
        const bool shaped = A.eos.shape != LBM_SHAPE_NONE, pr = A.eos.base == LBM_BASE_PR;
        if (nt) fd_launch<true>(pr, shaped, grd, s, A, c);
        else fd_launch<false>(pr, shaped, grd, s, A, c);
        if (!ok(hipGetLastError(), "fd step launch")) return LBM_EHIP;
        // the new state is in (rs, us, vs): swap the roles of the two state buffers
        std::swap(c->rho, c->rs);
        std::swap(c->u, c->us);
        std::swap(c->v, c->vs);
        c->step++;
    }
    return LBM_OK;
}

int lbm_fd_fields(lbm_fd_ctx* c, double* rho, double* u, double* v, void* stream)
{
    if (!c) return LBM_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    const size_t nb = c->n * sizeof(double);
    bool good = true;
    if (rho) good = good && ok(hipMemcpyAsync(rho, c->rho, nb, hipMemcpyDeviceToDevice, s), "fd rho out");
    if (u) good = good && ok(hipMemcpyAsync(u, c->u, nb, hipMemcpyDeviceToDevice, s), "fd u out");
    if (v) good = good && ok(hipMemcpyAsync(v, c->v, nb, hipMemcpyDeviceToDevice, s), "fd v out");
    return good ? LBM_OK : LBM_EHIP;
}

int lbm_fd_status(lbm_fd_ctx* c, void* stream)
{
    if (!c) return LBM_EINVAL;
    unsigned h[2];
    hipStream_t s = (hipStream_t)stream;
    if (!ok(hipMemcpyAsync(h, c->err, sizeof(h), hipMemcpyDeviceToHost, s), "fd status") ||
        !ok(hipStreamSynchronize(s), "fd status sync"))
        return LBM_EHIP;
    if (h[0]) {
        char buf[160];
        std::snprintf(buf, sizeof(buf), "lbm_fd: psi^2 < 0 or non-positive density at step %u", h[1]);
        lbm_set_error(buf);
        return LBM_EUNSTABLE;
    }
    return LBM_OK;
}

void lbm_fd_destroy(lbm_fd_ctx* c) { delete c; }

}  // extern "C"
