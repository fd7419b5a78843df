// The 2D right-hand side of one tile and its Runge-Kutta stage combination,
// shared by the single-grid kernel (plane.hip) and the batched one
// (batch.hip).
//
// A workgroup of 512 threads owns a TX x TY tile.  Its first 256 threads take
// the x sweep and its last 256 the y sweep, at the same time: one thread per
// reconstruction of its direction (the tile's cells and one halo cell per
// side), which then solves the face on the reconstruction's + side with its
// own + values in registers, so that only the - values and the fluxes pass
// through LDS.  The tile's sizes keep every phase to a single pass of the 256
// threads.  At the end both halves hold the tile's cells and share the
// variables: the y half forms rows 0 .. 2, the x half, which converted the
// cells, the momentum in y, the energy and alpha1 with its source.  Three
// barriers per tile.
//
// What it is bound by: the latency of one wavefront's chain on a grid of a
// few hundred tiles (one run), instruction issue on many (an ensemble).  The
// first halves with the two sweeps side by side, the second gained from the
// single pass: a 16 x 16 tile's 288 reconstructions took two passes of 256
// threads, the second one-eighth full.
//
// 253 x 181 cells FP64 (208 tiles): 8.0 us a launch, 11.5 with one sweep after
// the other on 256 threads.  30285 tiles of the 64 .. 512 ensemble in FP32:
// 286 us a launch, 332 so (about 800 issue slots per wavefront and tile: within
// a few percent of the card's issue rate).
#pragma once

#include "charbc.h"
#include "internal.h"
#include "mlp.h"

namespace mfc {

template <int TX_, int TY_>
struct Tile2 {
    static constexpr int TX = TX_, TY = TY_, NV = 6, E = 4, A = 5;
    static constexpr int NS = 256, NT = 2 * NS;         // threads of one sweep, of the workgroup
    static constexpr int PX = TX + 2 * NG, PY = TY + 2 * NG;
    static constexpr int NPX = (TX + 2) * TY, NPY = TX * (TY + 2);  // reconstructions of a sweep
    static constexpr int NOWN = TX * TY, NHALO = 2 * NG * (TX + TY);
    static_assert(NPX <= NS && NPY <= NS && NOWN <= NS && NHALO <= NS, "one pass of a sweep's threads per phase");
};

template <class T, class S>
struct Tile2Lds {
    T plane[S::NV][S::PY][S::PX];
    T minus[2][S::NV][S::NS];       // - face value of every reconstruction, per sweep
    T flux[2][S::NV + 1][S::NS];    // flux and face velocity of the face above every reconstruction
};

// This thread's role in a tile.
template <class S>
struct Role2 {
    int sweep, p;         // 0: x sweep, 1: y sweep; index within it
    int lx, ly;           // cell of the tile's window this thread converts, from the tile's first cell
    bool loads;           // whether there is one (x half: the tile's cells, y half: the halo)
    __device__ __forceinline__ Role2()
    {
        sweep = __builtin_amdgcn_readfirstlane((int)threadIdx.x / S::NS);   // whole wavefronts
        p = (int)threadIdx.x % S::NS;
        if (sweep == 0) {
            loads = p < S::NOWN;
            lx = p % S::TX;
            ly = p / S::TX;
        } else {
            loads = p < S::NHALO;
            if (p < 2 * NG * S::TY) {
                const int c = p % (2 * NG);
                lx = c < NG ? c - NG : S::TX + c - NG;
                ly = p / (2 * NG);
            } else {
                const int h = p - 2 * NG * S::TY, r = h / S::TX;
                lx = h % S::TX;
                ly = r < NG ? r - NG : S::TY + r - NG;
            }
        }
    }
};

// States are in global memory: said where the compiler cannot see it (pointers
// that are themselves read from memory), which would give flat accesses.
template <class T>
using Global = __attribute__((address_space(1))) T;

// Whether the window of the tile at (x0, y0) lies in the interior.
template <class S>
__device__ __forceinline__ bool inner2(const Grid &g, int x0, int y0)
{
    return x0 >= NG && y0 >= NG && x0 + S::TX + NG <= g.n[0] && y0 + S::TY + NG <= g.n[1];
}

// Conservative values of cell (i, j), clamped into the padded grid (cells
// past a ragged tile edge load a duplicate whose results are discarded).
// by_rule: neighbours past a face through the boundary rule (bc_cell: the
// values a ghost fill would write, bit for bit), otherwise from the ghost
// cells.  Returns whether the cell is one the method reads (an edge or corner
// ghost cell, which is never written, must not raise the flag).
// inner: the whole window lies in the interior (the same for all threads).
template <class T>
__device__ __forceinline__ bool load_cell2(const Grid &g, const T *q, int i, int j, bool by_rule, bool inner, T *qc)
{
    if (inner) {
        const Global<T> *src = (const Global<T> *)q + (int64_t)(j + NG) * g.stride[1] + (i + NG);
#pragma unroll
        for (int v = 0; v < 6; v++) qc[v] = src[v * g.vstride];
        return true;
    }
    i = min(i, g.n[0] + NG - 1);
    j = min(j, g.n[1] + NG - 1);
    const bool read = (i >= 0 && i < g.n[0]) || (j >= 0 && j < g.n[1]);
    if (by_rule) {
        i = bc_cell(i, g.n[0], g.bc[0], g.bc[1]);
        j = bc_cell(j, g.n[1], g.bc[2], g.bc[3]);
    }
    const Global<T> *src = (const Global<T> *)q + (int64_t)(j + NG) * g.stride[1] + (i + NG);
#pragma unroll
    for (int v = 0; v < 6; v++) qc[v] = src[v * g.vstride];
    return read;
}

// max_d |u_d| + c of a stored state (over dx_d on non-uniform cells, i and j
// its cell), the quantity of the CFL condition (Sec. 1), as the wave-speed
// kernels form it from the stored values.
template <class T, bool STRETCH>
__device__ __forceinline__ double signal2(const Grid &g, const T *qc, int i, int j)
{
    T w[6];
    cons_to_prim<2, T>(g, qc, w);
    double Gam, Pi;
    mixture<double>(g, double(w[5]), Gam, Pi);
    const double cs = sqrtT(sound2<double>(Gam, Pi, double(w[0]) + double(w[1]), double(w[4])));
    const double ax = __builtin_fabs(double(w[2])), ay = __builtin_fabs(double(w[3]));
    if constexpr (STRETCH) return __builtin_fmax((ax + cs) * inv_width(g, 0, i), (ay + cs) * inv_width(g, 1, j));
    else return __builtin_fmax(ax, ay) + cs;
}

// Characteristic rates (charbc.h, Sec. 3.3) of the boundary cell at plane
// position (r, c) on face SIDE of dimension D, from the cell and the next two
// cells into the domain.
template <int D, int SIDE, class T, int PY, int PX>
__device__ __forceinline__ bool tile2_char_rate(const Grid &g, const T (&pl)[6][PY][PX], int r, int c, T inv_dx, T *rate)
{
    constexpr int sg = SIDE == 0 ? 1 : -1;
    T W[3][6];
#pragma unroll
    for (int j = 0; j < 3; j++)
#pragma unroll
        for (int v = 0; v < 6; v++) W[j][v] = D == 0 ? pl[v][r][c + sg * j] : pl[v][r + sg * j][c];
    return char_rate<2, D, SIDE, T>(g, W[0], W[1], W[2], inv_dx, one_sided<T>(g, D, SIDE), rate);
}

// One variable group of a cell's stage result: rows V0 .. V0 + 2 from the
// faces around it.  fx, fy: its low x and y faces; rx (if hx), ry (if hy):
// characteristic rates in place of its x or y terms.  The sum of a cell
// without them is written as one fused product each, so that it is rounded
// alike with and without the rates in the kernel.
template <int V0, class T, class S>
__device__ __forceinline__ void combine2(const Tile2Lds<T, S> &L, int fx, int fy, T idx, T idy, bool hx, const T *rx,
                                         bool hy, const T *ry, T hsrc, T *out)
{
#pragma unroll
    for (int k = 0; k < 3; k++) {
        const int v = V0 + k;
        const T dx = L.flux[0][v][fx] - L.flux[0][v][fx + 1];
        const T dy = L.flux[1][v][fy] - L.flux[1][v][fy + S::TX];
        out[k] = fmaT(dx, idx, dy * idy);
        if (hx || hy) out[k] = (hx ? rx[v] : dx * idx) + (hy ? ry[v] : dy * idy);
    }
    if constexpr (V0 + 2 == S::A) {
        const T dx = L.flux[0][S::NV][fx + 1] - L.flux[0][S::NV][fx];
        const T dy = L.flux[1][S::NV][fy + S::TX] - L.flux[1][S::NV][fy];
        T divu = fmaT(dx, idx, dy * idy);
        if (hx || hy) divu = (hx ? T(0) : dx * idx) + (hy ? T(0) : dy * idy);
        out[2] = fmaT(hsrc, divu, out[2]);
    }
}

// The tile whose first cell is (x0, y0), from this thread's converted cell
// `qc` (loaded by load_cell2; `read` its return value).  `prefetch` issues the
// next tile's load.  mode 0: out = the right-hand side; mode 1, 2, 3: the
// SSP-RK3 stage combination (Sec. 3.4) of q0 and q with the step size hdt().
// `speed`: returns the wave speed of this thread's cell of the result (the
// caller reduces it; every thread calls with the same value).
template <class T, class S, bool ROUTE, int ORDER, bool STRETCH, bool CHAR, class Prefetch, class Dt>
__device__ __forceinline__ double tile2_stage(const Grid &g, Tile2Lds<T, S> &L, const Role2<S> &R, int x0, int y0,
                                              const T (&qc)[6], bool read, const T *q, const T *q0, T *out, int mode,
                                              bool speed, bool &bad, const mlp::Params *net, uint16_t *scratch,
                                              float logit_tau, T sqrt_eps, Prefetch prefetch, Dt step_size)
{
    constexpr int NV = S::NV, E = S::E, A = S::A, TX = S::TX, TY = S::TY;
    const T eps = T(g.eps);
    const int p = R.p;
    if (R.loads) {
        T w[NV];
        bad |= cons_to_prim<2, T>(g, qc, w) && read;
#pragma unroll
        for (int v = 0; v < NV; v++) L.plane[v][R.ly + NG][R.lx + NG] = w[v];
    }
    __syncthreads();
    prefetch();

    // reconstruct cell p % (TX + 2) - 1 of row p / (TX + 2) along x, or row
    // p / TX - 1 of column p % TX along y
    const int np = R.sweep == 0 ? S::NPX : S::NPY, step = R.sweep == 0 ? 1 : S::PX;
    const int width = R.sweep == 0 ? TX + 2 : TX;
    const bool rec = p < np;
    const int pc = rec ? p : np - 1, row = pc / width, col = pc % width;
    const int r0 = R.sweep == 0 ? row + NG : row, c0 = R.sweep == 0 ? col : col + NG;   // first stencil cell
    T wP[NV];
    bool lin = false;
    if constexpr (ROUTE) {   // whole wavefronts classify together
        if (__ballot(rec))
            lin = mlp::smooth_stencil<T>(*net, scratch, &L.plane[A][r0][c0], &L.plane[0][r0][c0], &L.plane[1][r0][c0],
                                         &L.plane[E][r0][c0], step, sqrt_eps, logit_tau, (int)threadIdx.x % 64);
    }
    if (rec) {
        const double *cf = STRETCH ? coef_row(g, R.sweep, R.sweep == 0 ? x0 + col - 1 : y0 + row - 1) : nullptr;
#pragma unroll
        for (int v = 0; v < NV; v++) {
            const T *s = &L.plane[v][r0][c0];
            T &m = L.minus[R.sweep][v][p];
            if (ROUTE && lin) linear5_pair<T>(s[0], s[step], s[2 * step], s[3 * step], s[4 * step], wP[v], m);
            else recon_cell<ORDER, T>(cf, s[0], s[step], s[2 * step], s[3 * step], s[4 * step], eps, wP[v], m);
        }
    }
    __syncthreads();

    // this thread's cell of the result, and the operands of its combination
    const int tx = p % TX, ty = p / TX, gx = x0 + tx, gy = y0 + ty;
    const bool own = p < S::NOWN && gx < g.n[0] && gy < g.n[1];
    const int v0 = R.sweep == 0 ? 3 : 0;
    const int64_t c = (int64_t)(gy + NG) * g.stride[1] + (gx + NG);
    T a0[3], a1[3];
    if (own && mode != 0) {
#pragma unroll
        for (int k = 0; k < 3; k++) {
            a1[k] = ((const Global<T> *)q)[(v0 + k) * g.vstride + c];
            a0[k] = mode == 1 ? a1[k] : ((const Global<T> *)q0)[(v0 + k) * g.vstride + c];
        }
    }

    // faces: above reconstruction p in x (col <= TX), in y (row <= TY)
    {
        T wR[NV], F[NV], uf;
        if (R.sweep == 0) {
            if (rec && col <= TX) {
#pragma unroll
                for (int v = 0; v < NV; v++) wR[v] = L.minus[0][v][p + 1];
                const bool b = hllc<2, 0, T>(g, wP, wR, F, uf);
                bad |= b && (y0 + row < g.n[1]) && (x0 + col <= g.n[0]);
#pragma unroll
                for (int v = 0; v < NV; v++) L.flux[0][v][p] = F[v];
                L.flux[0][NV][p] = uf;
            }
        } else if (rec && row <= TY) {
#pragma unroll
            for (int v = 0; v < NV; v++) wR[v] = L.minus[1][v][p + TX];
            const bool b = hllc<2, 1, T>(g, wP, wR, F, uf);
            bad |= b && (x0 + col < g.n[0]) && (y0 + row <= g.n[1]);
#pragma unroll
            for (int v = 0; v < NV; v++) L.flux[1][v][p] = F[v];
            L.flux[1][NV][p] = uf;
        }
    }
    __syncthreads();

    T r[3];
    if (own) {
        const T idx = STRETCH ? T(inv_width(g, 0, gx)) : T(g.inv_dx[0]);
        const T idy = STRETCH ? T(inv_width(g, 1, gy)) : T(g.inv_dx[1]);
        const int fx = ty * (TX + 2) + tx, fy = ty * TX + tx;
        bool hx = false, hy = false;
        T xrate[NV], yrate[NV];
        if constexpr (CHAR) {   // boundary cells of characteristic faces take their rates in place of the normal terms
            const int pr = ty + NG, pcx = tx + NG;
            if (gx == 0 && g.bc[0] == MFC_BC_CHARACTERISTIC) bad |= tile2_char_rate<0, 0>(g, L.plane, pr, pcx, idx, xrate), hx = true;
            else if (gx == g.n[0] - 1 && g.bc[1] == MFC_BC_CHARACTERISTIC) bad |= tile2_char_rate<0, 1>(g, L.plane, pr, pcx, idx, xrate), hx = true;
            if (gy == 0 && g.bc[2] == MFC_BC_CHARACTERISTIC) bad |= tile2_char_rate<1, 0>(g, L.plane, pr, pcx, idy, yrate), hy = true;
            else if (gy == g.n[1] - 1 && g.bc[3] == MFC_BC_CHARACTERISTIC) bad |= tile2_char_rate<1, 1>(g, L.plane, pr, pcx, idy, yrate), hy = true;
        }
        if (R.sweep == 0) {
            // the source coefficient from the cell's own slot, which this thread wrote
            const T hsrc = alpha_source<T>(g, L.plane[A][ty + NG][tx + NG], L.plane[E][ty + NG][tx + NG]);
            combine2<3, T, S>(L, fx, fy, idx, idy, hx, xrate, hy, yrate, hsrc, r);
        } else {
            combine2<0, T, S>(L, fx, fy, idx, idy, hx, xrate, hy, yrate, T(0), r);
        }
        if (mode != 0) {
            const T hdt = T(step_size());
            const T ca = T(mode == 1 ? 0.0 : (mode == 2 ? 0.75 : 1.0 / 3.0));
            const T cb = T(mode == 1 ? 1.0 : (mode == 2 ? 0.25 : 2.0 / 3.0));
#pragma unroll
            for (int k = 0; k < 3; k++) r[k] = ca * a0[k] + cb * (a1[k] + hdt * r[k]);
        }
#pragma unroll
        for (int k = 0; k < 3; k++) ((Global<T> *)out)[(v0 + k) * g.vstride + c] = r[k];
    }
    // The next tile writes plane before its first barrier (the reads above,
    // of a thread's own slot alone, are past; with characteristic faces
    // neighbours' slots are read too and the tile ends on a barrier), minus
    // and flux after it.
    double sp = 0.0;
    if (speed) {   // the y half hands its rows over (minus was last read before the third barrier)
        if (own && R.sweep == 1) {
#pragma unroll
            for (int k = 0; k < 3; k++) L.minus[0][k][p] = r[k];
        }
        __syncthreads();
        if (own && R.sweep == 0) {
            const T full[6] = {L.minus[0][0][p], L.minus[0][1][p], L.minus[0][2][p], r[0], r[1], r[2]};
            sp = signal2<T, STRETCH>(g, full, gx, gy);
        }
    } else if constexpr (CHAR) {
        if (g.bc[0] == MFC_BC_CHARACTERISTIC || g.bc[1] == MFC_BC_CHARACTERISTIC || g.bc[2] == MFC_BC_CHARACTERISTIC ||
            g.bc[3] == MFC_BC_CHARACTERISTIC)
            __syncthreads();
    }
    return sp;
}

}  // namespace mfc
