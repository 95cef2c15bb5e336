// Many time steps per launch for short periodic lattices, the populations kept in LDS between
// them (included by lbm_step.hip and lbm_batched.hip).
//
// A workgroup holds every row of `cols` columns of its lattice, one node per thread, and
// advances them `nsteps` steps: the first pull reads HBM, the later ones read the
// post-collision populations of the neighbours from LDS, and the last step stores.  Rows wrap
// inside the workgroup.  A lattice of at most `cols` columns wraps there in x too (resident:
// any number of steps per launch); a wider one is cut into strips, each grown on both sides
// by the columns that the steps of a launch use up: one node per pull and one per
// Eq. ShanChenForce stencil, 2 n - 1 for n steps (the last force reaches the strip's edge).
//
// What bounds it: one workgroup's latency (two barriers, two LDS round trips and a chain of
// about 220 FP64 or 150 FP32 vector instructions per step), not memory: the lattice is read
// and written once per launch.  Two steps per launch, the general path's way, spend most of
// their time in the launch and its loads at these sizes.
#pragma once

#include "lbm_device.h"

namespace lbmk {

constexpr int kStripMaxRows = 16;      // tallest lattice cut into strips
constexpr int kStripThreads = 1024;    // most nodes of a workgroup
constexpr int kResidentSteps = 4096;   // most steps per launch of resident lattices

// How the strip kernel runs a set of lattices: threads of its workgroups and steps per launch
// (0 threads: it does not; kResidentSteps: every lattice is resident)
struct StripPlan {
    int threads, steps;
};
inline int strip_halo(int steps) { return 2 * steps - 1; }
// columns that a workgroup holds of lattice p (its width: resident), and those it advances in a
// launch of `steps` steps
inline int strip_cols(const lbm_params& p, int threads)
{
    const int c = threads / p.ny;
    return c < p.nx ? c : p.nx;
}
inline int strip_out(const lbm_params& p, int threads, int steps)
{
    const int c = strip_cols(p, threads);
    return c == p.nx ? c : c - 2 * strip_halo(steps);
}

// Lattices that fit: periodic, and short or small enough for one workgroup.  Among workgroup
// sizes and steps per launch the least estimated time per step is taken.  The estimate: a
// launch with its first loads and last stores (about 5 us beside the traffic), shared by its
// steps, and per step, with w the waves on a SIMD of the busiest CU (workgroups dealt out over
// 256 CUs), the latency of a step, 0.9 us + 0.15 w in FP32 and 0.5 us + 0.26 w in FP64, or the
// issue of its instructions, 0.38 w and 0.62 w, whichever is more.  Fitted to a sweep on
// MI355X over 64 to 1024 threads and 2 to 16 steps: single lattices of 1 to 16 rows and batches
// of 64 to 300; the choice came within 6% of the best of the sweep in each.
inline StripPlan strip_plan(int B, const lbm_params* p)
{
    const bool f32 = p[0].prec == LBM_FP32_SHIFTED;
    StripPlan best = {0, 0};
    bool all_resident = true;
    for (int b = 0; b < B; ++b) {
        if (p[b].walls || p[b].ny > kStripThreads) return best;
        const bool fits = (long long)p[b].nx * p[b].ny <= kStripThreads;
        if (!fits && p[b].ny > kStripMaxRows) return best;
        all_resident = all_resident && fits;
    }
    double best_us = 0.0;
    const int steps[] = {16, 12, 8, 6, 4, 2};
    // FP32 strips stay within 768 threads: at the kernel's 80 vector registers a CU holds two such
    // workgroups but one of more waves (300 lattices of 16 rows: 25 us/step in pairs, 32 alone)
    const int tmax = f32 && !all_resident ? 768 : kStripThreads;
    for (int t = 64; t <= tmax; t += 64) {
        for (int si = all_resident ? -1 : 0; si < (all_resident ? 0 : 6); ++si) {
            const int n = si < 0 ? kResidentSteps : steps[si];
            long long groups = 0, used = 0;
            double bytes = 0.0;
            bool ok = true;
            for (int b = 0; b < B && ok; ++b) {
                const int c = t / p[b].ny < 1 ? 0 : strip_cols(p[b], t);
                const int out = c == 0 || (si < 0 && c < p[b].nx) ? 0 : strip_out(p[b], t, n);
                ok = out >= 1 && (c == p[b].nx || (out >= 8 && p[b].nx > strip_halo(n)));
                if (!ok) break;
                const long long k = (p[b].nx + out - 1) / out;
                groups += k;
                used = c * p[b].ny > used ? c * p[b].ny : used;
                bytes += (double)k * (c + out) * p[b].ny * (f32 ? 40 : 72);
            }
            if (!ok) continue;
            const double waves = (double)((used + 63) / 64);
            const double w = (double)((groups + 255) / 256) * (waves < 4.0 ? 1.0 : waves / 4.0);
            const double latency = f32 ? 0.9 + 0.15 * w : 0.5 + 0.26 * w, issue = w * (f32 ? 0.38 : 0.62);
            const double us = (5.0 + bytes * 2e-7) / n + (issue > latency ? issue : latency);
            if (!best.threads || us < best_us) {
                best = {(int)waves * 64, n};
                best_us = us;
            }
        }
    }
    return best;
}

// The plan of a single lattice (lbm_init): of the automatic variant only, since an explicit one, or a
// named or timed tile height, runs what it names
inline StripPlan lattice_strip_plan(const lbm_params& p)
{
    return p.kernel_variant == LBM_VARIANT_AUTO && p.tile_rows == 0 ? strip_plan(1, &p) : StripPlan{0, 0};
}

// Whether a single lattice leaves a launch of `steps` steps to the strip kernel.  One and two steps
// run on the one- and two-step kernels, whose smaller workgroups take less time for so little work,
// except on wide lattices of so few rows that tiles of 10 and more are mostly empty and yet more
// than the chip has compute units.  Measured, us per call, strips / those kernels: one step 1024 x 1
// FP64 5.05 / 3.73, 2048 x 4 FP64 4.58 / 4.09, 1500 x 3 FP32 4.16 / 3.85, 4096 x 16 FP32 5.06 / 4.52,
// but 16384 x 4 FP64 5.1 / 5.7, 65536 x 1 FP32 4.3 / 6.4; two steps 1024 x 1 FP64 6.8 / 5.5, 700 x 12
// FP32 6.0 / 5.6, but 16384 x 4 FP64 6.6 / 8.4, 65536 x 1 FP32 5.6 / 10.7; three steps, where the other
// kernels take two launches, 1024 x 1 FP64 8.5 / 10.0, 4096 x 16 FP32 8.5 / 11.4.
inline bool strip_runs(const lbm_params& p, long long steps) { return steps > 2 || (p.ny <= 4 && p.nx >= 15000); }

template <typename T, int CAP>
struct StripLds {
    DevEos eos;
    T mv[8][CAP];            // post-collision moving populations of the last step
    T ps[CAP];
    double red[CAP / 64][3];  // a reducing launch's wave totals (mass, momentum)
};

// Advance columns x0 .. x0 + out - 1 (all rows) of lattice A by nsteps steps from src to dst,
// holding `cols` of them (all, or halo more on each side, halo >= 2 nsteps - 1); `step` is
// added to A.step for the number of the first step.  REDUCE: the last step leaves the FP64 mass and
// momentum of these columns in partial[0..2].  NT: streaming stores, for small lattices as in the
// other kernels (kStreamBytes).  Streamed, a larger lattice is no longer in the memory-side cache for
// the next launch: 65536 x 16, us for 100 steps (and for one), streamed / not, FP64 1833 / 1708 (47.1 /
// 38.9), FP32 991 / 941 (32.3 / 24.7).
template <typename T, int CAP, bool REDUCE, bool NT>
__device__ __forceinline__ void strip_steps(const StepArgs& A, const void* src, void* dst, int x0, int cols, int out,
                                            int halo, int nsteps, int step, double* partial, StripLds<T, CAP>& S)
{
    const int n = threadIdx.x;
    const int ny = A.ny, nx = A.nx;
    const int y = n / cols, c = n - y * cols;
    const bool resident = cols == nx;
    const int G = resident ? 0 : halo;
    const int W = min(out, nx - x0);
    // columns from the strip to this one; the steps of a launch use them up
    const int d = c < G ? G - c : (c > G + W - 1 ? c - (G + W - 1) : 0);
    const bool row = y < ny;
    // neighbours inside the workgroup: rows wrap, columns wrap when the lattice is resident
    const int dw = c > 0 ? -1 : (resident ? cols - 1 : 0), de = c + 1 < cols ? 1 : (resident ? 1 - cols : 0);
    const int ds = y > 0 ? -cols : (ny - 1) * cols, dn = y + 1 < ny ? cols : -(ny - 1) * cols;
    const int at = row ? n : 0;
    const int iw = at + (row ? dw : 0), ie = at + (row ? de : 0), is = at + (row ? ds : 0), in = at + (row ? dn : 0);
    const int isw = is + iw - at, ise = is + ie - at, inw = in + iw - at, ine = in + ie - at;
    int x = x0 - G + c;
    x = x < 0 ? x + nx : (x >= nx ? x - nx : x);
    Lane L;
    L.lane = n & 63;
    L.x = x;
    L.xm = x == 0 ? nx - 1 : x - 1;
    L.xp = x == nx - 1 ? 0 : x + 1;
    L.valid = L.interior = true;
    if (n == 0) S.eos = A.eos;
    Acc acc = {0.0, 0.0, 0.0};
    Row<T> R;
    R.g0 = 0.0;
#pragma unroll
    for (int i = 0; i < 9; ++i) R.g[i] = (T)0;
    if (row && d <= 2 * nsteps - 1) {
        const View<T> V = make_view<T>(src, A.plane);
        pull<T>(V, A, L.x, L.xm, L.xp, y, R.g0, R.g);
    }
    __syncthreads();
    for (int s = 0;; ++s) {
        const double dr = node_drho<T>(R.g0, R.g);
        const int left = nsteps - 1 - s;
        // columns beyond 2 left + 1 have used up their neighbours: whatever they hold is not read
        // by a column that has not, and is not checked
        const T ps = node_psi<T>(A, S.eos, A.eos.base, A.eos.shape, dr, row && d <= 2 * left + 1, step + s);
        S.ps[n] = ps;
        __syncthreads();
        T Ftx, Fty;
        force_tilde<T>(A, S.ps[isw], S.ps[is], S.ps[ise], S.ps[iw], S.ps[ie], S.ps[inw], S.ps[in], S.ps[ine], Ftx, Fty);
        T o[9];
        double o0;
        Acc a = {0.0, 0.0, 0.0};
        node_collide<T, REDUCE ? MODE_STEP_REDUCE : MODE_STEP>(A, L, y, R, dr, ps, Ftx, Fty, a, o, o0);
        if (left == 0) {
            if (row && d == 0) {
                acc = a;
                const WView<T> D = make_wview<T>(dst, A.plane);
                const uint32_t off = (uint32_t)y * (uint32_t)A.ld + (uint32_t)x;
                if constexpr (NT) {
#pragma unroll
                    for (int i = 1; i < 9; ++i)
                        __builtin_nontemporal_store(o[i], (T*)(D.mv[i] + off * (uint32_t)sizeof(T)));
                    __builtin_nontemporal_store(o0, (double*)(D.rest + off * 8u));
                } else {
#pragma unroll
                    for (int i = 1; i < 9; ++i) *(T*)(D.mv[i] + off * (uint32_t)sizeof(T)) = o[i];
                    *(double*)(D.rest + off * 8u) = o0;
                }
            }
            break;
        }
#pragma unroll
        for (int i = 1; i < 9; ++i) S.mv[i - 1][n] = o[i];
        __syncthreads();
        R.g0 = o0;
        R.g[1] = S.mv[0][iw];
        R.g[2] = S.mv[1][is];
        R.g[3] = S.mv[2][ie];
        R.g[4] = S.mv[3][in];
        R.g[5] = S.mv[4][isw];
        R.g[6] = S.mv[5][ise];
        R.g[7] = S.mv[6][ine];
        R.g[8] = S.mv[7][inw];
    }
    if (REDUCE) {
        const double m = wave_total(acc.m), jx = wave_total(acc.x), jy = wave_total(acc.y);
        const int w = n >> 6;
        if ((n & 63) == kTotalLane) {
            S.red[w][0] = m;
            S.red[w][1] = jx;
            S.red[w][2] = jy;
        }
        __syncthreads();
        if (n < 3) {
            double r = 0.0;
            for (int k = 0; k < (int)(blockDim.x >> 6); ++k) r += S.red[k][n];
            partial[n] = r;
        }
    }
}

}  // namespace lbmk
