// 1D runs of the fused kernel: whole SSP-RK3 steps (Sec. 3.4) in one launch.
//
// A 1D grid has work for a few wavefronts, so a run is the latency of its
// launches: eight per step with a ghost fill and a right-hand side per stage
// and the wave-speed reduction.  Here one thread per cell keeps its state in
// registers through the stages and exchanges primitives, face values and
// fluxes through LDS (three barriers per stage).
//   A grid of up to kLineMany cells is one workgroup, which takes many steps
// per launch: it reduces the wave speeds of its cells itself (up to kLineMax
// cells for a single step).
//   A longer one is cut into pieces that take one step per launch: a piece
// recomputes the nine cells on either side that its three stages reach (of 256
// positions 238 are kept), states go from buffer to buffer, and the step size
// comes from the maxima that the launch before left.
// Neighbours past a face are read through the boundary rule (bc_cell: the
// values a ghost fill would write, bit for bit).
//
// Ten steps FP64: 400 cells 82 us (the launches of before: 295), 250 cells 61
// (272), 4000 cells in pieces 100 (313).  Bound by the chain of one stage, 2.0
// us of 250 cells on the four SIMDs of one CU, 2.8 us of 400; beyond 512
// threads a workgroup's wavefronts queue on its CU and pieces, at 9.7 us a step
// with the launch, are the faster (700 cells: 97 us against 112).
#include <cmath>

#include "internal.h"

namespace mfc {
namespace {

constexpr int kPieceHalo = 9, kPieceThreads = 256, kPieceOwn = kPieceThreads - 2 * kPieceHalo;
constexpr int kLineThreads = 1024, kLineMax = kLineThreads - 2, kLineMany = 510;
constexpr int kLineSteps = 64;   // steps per launch of one workgroup (bounds a launch to a few ms)

struct LineRun {
    int steps;          // steps of this launch
    int halo, own;      // positions before a piece's first cell; cells per piece
    bool pieces;        // more than one workgroup
    bool ghosts;        // the last step's q^n goes to the ghost cells of `home`
    void *home;         // the caller's state
};

// One position's cell values, NT positions.
template <class T, int NT>
struct LineLds {
    T w[5][NT], minus[5][NT], flux[6][NT];
    double speed[NT / 64];
};

template <class T, int ORDER, bool STRETCH, int NT>
__global__ void __launch_bounds__(NT, NT / 256)
    k_line(Grid g, const T *q, T *out, LineRun run, StepSize ss, int *__restrict__ flag)
{
    constexpr int NV = 5, E = 3, A = 4;
    __shared__ LineLds<T, NT> L;
    const int n = g.n[0], p = threadIdx.x, nt = blockDim.x, waves = nt / 64;
    const int x0 = (int)blockIdx.x * run.own, base = x0 - run.halo, i = base + p;
    const bool wraps = run.pieces && g.bc[0] == MFC_BC_PERIODIC;   // positions past a face are copies of cells
    const bool inside = i >= 0 && i < n;
    const bool live = inside || (wraps && i < n + kPieceHalo);     // has a state
    const bool own = inside && i >= x0 && i < x0 + run.own;
    const bool one = blockIdx.x == 0 && p == 0;
    const int ic = wraps && live ? bc_cell(i, n, g.bc[0], g.bc[1]) : i;   // the cell a copy is of
    const T eps = T(g.eps), ix = STRETCH ? T(inv_width(g, 0, ic)) : T(g.inv_dx[0]);
    const double *cf = STRETCH ? coef_row(g, 0, ic) : nullptr;
    // position of each cell of this position's stencil
    int st[5];
#pragma unroll
    for (int k = 0; k < 5; k++) {
        int j = i + k - 2;
        if (!wraps) j = bc_cell(j, n, g.bc[0], g.bc[1]);
        st[k] = min(max(j - base, 0), nt - 1);
    }
    const int64_t c = (live ? ic : 0) + NG;
    T qs[NV], q0[NV], w[NV];
#pragma unroll
    for (int v = 0; v < NV; v++) qs[v] = q[v * g.vstride + c];
    bool bad = false;
    double h = 0.0, t = ss.scalars[2], m = 0.0;
    if (run.pieces && ss.speeds) {   // gathered by the first barrier
        const double a = ss.gather(nt);
        if (p % 64 == 0) L.speed[p / 64] = a;
    }

    // max (|u| + c) of the cell, as the wave-speed kernel forms it
    auto signal = [&] {
        double Gam, Pi;
        mixture<double>(g, double(w[A]), Gam, Pi);
        const double cs = sqrtT(sound2<double>(Gam, Pi, double(w[0]) + double(w[1]), double(w[E])));
        const double a = __builtin_fabs(double(w[2])) + cs;
        return STRETCH ? a * inv_width(g, 0, i) : a;
    };

    for (int step = 0; step < run.steps; step++) {
        if (run.ghosts && step + 1 == run.steps && own) {   // as a fill of q^n leaves them
            T *home = (T *)run.home;
            const bool periodic = g.bc[0] == MFC_BC_PERIODIC;
#pragma unroll
            for (int v = 0; v < NV; v++) {
                T *row = home + v * g.vstride + NG;
                if (periodic) {
                    if (i < NG) row[n + i] = qs[v];
                    if (i >= n - NG) row[i - n] = qs[v];
                } else {
#pragma unroll
                    for (int l = 1; l <= NG; l++) {
                        if (i == 0) row[-l] = qs[v];
                        if (i == n - 1) row[n - 1 + l] = qs[v];
                    }
                }
            }
        }
#pragma unroll
        for (int v = 0; v < NV; v++) q0[v] = qs[v];
#pragma unroll 1
        for (int mode = 1; mode <= 3; mode++) {
            if (live) {
                const bool b = cons_to_prim<1, T>(g, qs, w);
                bad |= b && own;
#pragma unroll
                for (int v = 0; v < NV; v++) L.w[v][p] = w[v];
            }
            if (mode == 1 && !run.pieces && ss.cfl > 0.0) {
                const double a = wave_max(own ? signal() : 0.0);
                if (p % 64 == 0) L.speed[p / 64] = a;
            }
            __syncthreads();
            if (mode == 1) {
                if (ss.cfl > 0.0 && (!run.pieces || ss.speeds)) {
                    m = 0.0;
                    for (int k = 0; k < waves; k++) m = __builtin_fmax(m, L.speed[k]);
                    h = ss.cfl * ss.dxmin / m;
                } else {
                    h = ss.set ? ss.dt : ss.scalars[1];
                }
                t += h;
            }
            T wP[NV];
#pragma unroll
            for (int v = 0; v < NV; v++)
                recon_cell<ORDER, T>(cf, L.w[v][st[0]], L.w[v][st[1]], L.w[v][st[2]], L.w[v][st[3]], L.w[v][st[4]], eps,
                                     wP[v], L.minus[v][p]);
            __syncthreads();
            // the face between this position and the next
            T F[NV], uf, wR[NV];
#pragma unroll
            for (int v = 0; v < NV; v++) wR[v] = L.minus[v][min(p + 1, nt - 1)];
            const bool b = hllc<1, 0, T>(g, wP, wR, F, uf);
            bad |= b && i >= x0 - 1 && i < min(x0 + run.own, n);   // a face of an own cell
            // the face's values as rounded before any use: the cell above takes them from LDS
#pragma unroll
            for (int v = 0; v < NV; v++) {
                __asm__ volatile("" : "+v"(F[v]));
                L.flux[v][p] = F[v];
            }
            __asm__ volatile("" : "+v"(uf));
            L.flux[NV][p] = uf;
            __syncthreads();
            if (live) {
                const int lo = max(p - 1, 0);
                const T hdt = T(h);
                const T ca = T(mode == 1 ? 0.0 : (mode == 2 ? 0.75 : 1.0 / 3.0));
                const T cb = T(mode == 1 ? 1.0 : (mode == 2 ? 0.25 : 2.0 / 3.0));
                T D[NV];
#pragma unroll
                for (int v = 0; v < NV; v++) D[v] = (L.flux[v][lo] - F[v]) * ix;
                const T divu = (uf - L.flux[NV][lo]) * ix;
                D[A] += alpha_source<T>(g, w[A], w[E]) * divu;
#pragma unroll
                for (int v = 0; v < NV; v++) qs[v] = ca * q0[v] + cb * (qs[v] + hdt * D[v]);
            }
        }
    }
    if (own) {
#pragma unroll
        for (int v = 0; v < NV; v++) out[v * g.vstride + c] = qs[v];
    }
    if (ss.carry) {   // pieces: the next step's maxima, one per wavefront
        double a = 0.0;
        if (own) {
            cons_to_prim<1, T>(g, qs, w);
            a = signal();
        }
        a = wave_max(a);
        if (p % 64 == 0) ss.carry[blockIdx.x * waves + p / 64] = a;
    }
    if (one) {
        if (ss.cfl > 0.0 && (!run.pieces || ss.speeds)) ss.scalars[0] = m;
        if (!run.pieces || ss.set) {
            ss.scalars[1] = h;
            ss.scalars[2] = t;
            if (ss.dt_out) *ss.dt_out = h;
        }
    }
    if (bad) raise_flag(flag, 1);
}

template <class T, int ORDER, bool STRETCH>
int line_launch(mfc_grid *h, const void *q, void *out, const LineRun &run, const StepSize &ss, hipStream_t s)
{
    const Grid &g = h->g;
    if (run.pieces) {
        hipLaunchKernelGGL((k_line<T, ORDER, STRETCH, kPieceThreads>), dim3((g.n[0] + kPieceOwn - 1) / kPieceOwn),
                           dim3(kPieceThreads), 0, s, g, (const T *)q, (T *)out, run, ss, h->flag);
    } else {
        // the fewest threads that hold the grid: 1024 leave 128 registers each and spill
        const dim3 threads((g.n[0] + 2 + 63) / 64 * 64);
        auto one = [&](auto nt) {
            hipLaunchKernelGGL((k_line<T, ORDER, STRETCH, decltype(nt)::value>), dim3(1), threads, 0, s, g, (const T *)q,
                               (T *)out, run, ss, h->flag);
        };
        if (threads.x <= 256) one(std::integral_constant<int, 256>{});
        else if (threads.x <= 512) one(std::integral_constant<int, 512>{});
        else one(std::integral_constant<int, kLineThreads>{});
    }
    return hip_status(hipGetLastError(), "1D step launch");
}

template <class T>
int line_launch_t(mfc_grid *h, const void *q, void *out, const LineRun &run, const StepSize &ss, hipStream_t s)
{
    const int recon = h->desc.recon;
    if (h->g.stretched)
        return recon == MFC_RECON_FIRST_ORDER ? line_launch<T, 1, true>(h, q, out, run, ss, s)
                                              : line_launch<T, 5, true>(h, q, out, run, ss, s);
    switch (recon) {
    case MFC_RECON_WENO3: return line_launch<T, 3, false>(h, q, out, run, ss, s);
    case MFC_RECON_FIRST_ORDER: return line_launch<T, 1, false>(h, q, out, run, ss, s);
    default: return line_launch<T, 5, false>(h, q, out, run, ss, s);
    }
}

int launch(mfc_grid *h, const void *q, void *out, const LineRun &run, const StepSize &ss, hipStream_t s)
{
    return h->desc.precision == MFC_FP32_MIXED ? line_launch_t<float>(h, q, out, run, ss, s)
                                               : line_launch_t<double>(h, q, out, run, ss, s);
}

// Wave-speed maxima of a launch of pieces, one per wavefront.
int64_t piece_speeds(const Grid &g)
{
    return (int64_t)((g.n[0] + kPieceOwn - 1) / kPieceOwn) * (kPieceThreads / 64);
}
int64_t line_partials_half(const Grid &g) { return std::max<int64_t>(kReduceBlocks, piece_speeds(g)); }

}  // namespace

int64_t line_partials(const Grid &g) { return 2 * line_partials_half(g); }

// Neither the routed reconstruction, which classifies whole wavefronts, nor
// characteristic faces, whose boundary pass follows every stage, nor the
// timing of single right-hand sides; a lone step of a long grid would need a
// copy back.
//   A lone step of up to 1022 cells is one workgroup of up to 1024 threads,
// whose 128 registers each spill (FP64 WENO5 24, which costs little: 1022 cells
// 22 us against 37 of the launches per stage; 62 on non-uniform cells, FP32
// there 24).  Non-uniform WENO5 cells pass the launches, 47 us FP64 and 45
// FP32, at 638 and 702 cells (50 and 46; 574 and 638: 46 and 43; 1022: 71 and
// 61), so a lone step of more than 574 or 638 takes those.
bool takes_line(const mfc_grid *h, int nsteps)
{
    const bool coefficients = h->g.stretched && h->desc.recon == MFC_RECON_WENO5;
    const int lone = coefficients ? (h->desc.precision == MFC_FP64 ? 574 : 638) : kLineMax;
    return h->desc.kernel == MFC_KERNEL_FUSED && h->desc.ndim == 1 && h->desc.recon != MFC_RECON_LEARNED &&
           !has_cbc(h) && !h->timing && (nsteps > 1 || h->g.n[0] <= lone);
}

int run_line(mfc_grid *h, void *q, int nsteps, double cfl, double dt, double *dt_out, hipStream_t s)
{
    int st = MFC_OK;
    StepSize ss;
    ss.cfl = cfl;
    ss.dt = dt;
    ss.dxmin = h->g.dxmin;
    ss.scalars = h->scalars;
    ss.set = true;
    ss.dt_out = dt_out;
    LineRun run{};
    run.home = q;
    if (h->g.n[0] <= (nsteps > 1 ? kLineMany : kLineMax)) {
        run.halo = 1;
        run.own = h->g.n[0];
        for (int done = 0; done < nsteps && st == MFC_OK; done += run.steps) {
            run.steps = std::min(nsteps - done, kLineSteps);
            run.ghosts = done + run.steps == nsteps;
            st = launch(h, q, q, run, ss, s);
        }
        return st;
    }
    // pieces: from q through the stage registers and back (two steps, the last
    // three of an odd number)
    constexpr int kInStep = 2048;   // more maxima are reduced by their own launch, as for 2D
    const int64_t half = line_partials_half(h->g);   // a launch reads one half and writes the other
    run.pieces = true;
    run.steps = 1;
    run.halo = kPieceHalo;
    run.own = kPieceOwn;
    void *at = q, *A = h->stage_a, *B = h->stage_b;
    for (int k = 0; k < nsteps && st == MFC_OK; k++) {
        const int left = nsteps - k;   // steps from here on, this one included
        void *to = left == 1 ? q : (at == A ? (left % 2 == 0 ? B : q) : A);
        run.ghosts = left == 1;
        double *speeds = h->partial + (k & 1) * half;
        ss.carry = cfl > 0.0 && left > 1 ? h->partial + (~k & 1) * half : nullptr;
        if (cfl > 0.0) {
            ss.nspeeds = k > 0 ? (int)piece_speeds(h->g) : kReduceBlocks;
            if (k == 0) st = launch_wavespeed(h, q, s);
            const bool own_launch = ss.nspeeds > kInStep;
            ss.set = !own_launch;
            ss.speeds = own_launch ? nullptr : speeds;
            if (st == MFC_OK && own_launch) launch_step_begin(h, speeds, ss.nspeeds, cfl, 0.0, s);
        }
        if (st == MFC_OK) st = launch(h, at, to, run, ss, s);
        at = to;
    }
    return st;
}

}  // namespace mfc
