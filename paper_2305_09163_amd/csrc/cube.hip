// Steps on small 3D grids of the split path: a whole stage in one launch.
//
// A grid of a few hundred tiles leaves most of the chip idle and a stage is
// the latency of its two launches, each a chain of load, conversion,
// reconstruction and Riemann solve per direction.  Here a workgroup owns a
// 16 x 10 tile of one plane and takes the three sweeps side by side: three
// wavefronts along x, three along y and eight along z, one thread per
// reconstruction (of the three planes whose cells a cell's two z faces need),
// which then solves the face on its + side.  A cell's z planes are converted
// again by the workgroups above and below it and its z reconstructions are
// formed three times over, 1.7 times the work of the split kernels, which pays
// while the launch is one round of the chip (one 133 KB FP64 workgroup per CU).
#include <cmath>

#include "internal.h"

namespace mfc {
namespace {

constexpr int TX = 16, TY = 10, NOWN = TX * TY, NV = 7, E = 5, A = 6;
constexpr int PX = TX + 2 * NG, PY = TY + 2 * NG, PLANE = PX * PY;
constexpr int NZ = 2 * NG + 1;                        // planes of a cell's z stencils
constexpr int NPX = (TX + 2) * TY, NPY = TX * (TY + 2), NPZ = 3 * NOWN;
constexpr int Y0 = 192, Z0 = 384, NT = 896;           // first thread of the y and z sweeps
static_assert(NPX <= Y0 && NPY <= Z0 - Y0 && NPZ <= NT - Z0, "one pass of a sweep's threads per phase");
// cells to convert: the other planes of every column, the tile, its halo
constexpr int kOther = (NZ - 1) * NOWN, kTile = kOther + NOWN, kCells = kTile + 2 * NG * (TX + TY);
static_assert(kCells > NT && kCells <= 2 * NT, "two cells per thread");
constexpr int kResults = NV * NOWN;                   // (cell, variable) results
static_assert(kResults > NT && kResults <= 2 * NT, "two results per thread");

// LDS: the plane with its halos, then the columns (planes k - 3 .. k + 3),
// whose area the fluxes take over once the reconstructions are formed.
template <class T>
struct Lds {
    T plane[NV * PLANE];
    union {
        T column[NV * NZ * NOWN];
        T flux[(NV + 1) * NT];
    };
    T minus[NV * NT];
    double speed[NT / 64];
};

template <class T, int ORDER>
__global__ void __launch_bounds__(NT, 4)
    k_cube(Grid g, const T *__restrict__ q, const T *q0, T *out, int mode, StepSize ss, int tiles_x, int tiles_y,
           int *__restrict__ flag)
{
    __shared__ Lds<T> L;
    const int t = threadIdx.x;
    const int x0 = (int)(blockIdx.x % tiles_x) * TX, y0 = (int)(blockIdx.x / tiles_x % tiles_y) * TY;
    const int k = (int)(blockIdx.x / tiles_x / tiles_y);
    bool bad = false;
    if (ss.speeds) {   // gathered by the first barrier
        const double m = ss.gather(NT);
        if (t % 64 == 0) L.speed[t / 64] = m;
    }

    // ---- cells as primitives; positions past the domain through the boundary
    // rule, past a ragged tile edge duplicates whose results are discarded
    {
        T qc[2][NV];
        int at[2], col[2];   // plane and column slots (-1: none)
#pragma unroll
        for (int j = 0; j < 2; j++) {
            const int c = t + j * NT;
            at[j] = col[j] = -1;
            if (c >= kCells) continue;
            int lx, ly, z = k;
            if (c < kTile) {
                const int cell = c % NOWN, pl = c / NOWN;   // planes k - 3 .. k - 1, k + 1 .. k + 3, then k
                lx = cell % TX;
                ly = cell / TX;
                const int slot = pl == NZ - 1 ? NG : (pl < NG ? pl : pl + 1);
                z = k + slot - NG;
                col[j] = slot * NOWN + cell;
                if (slot == NG) at[j] = (ly + NG) * PX + lx + NG;
            } else {
                const int h = c - kTile;
                if (h < 2 * NG * TY) {
                    const int a = h % (2 * NG);
                    lx = a < NG ? a - NG : TX + a - NG;
                    ly = h / (2 * NG);
                } else {
                    const int r = (h - 2 * NG * TY) / TX;
                    lx = (h - 2 * NG * TY) % TX;
                    ly = r < NG ? r - NG : TY + r - NG;
                }
                at[j] = (ly + NG) * PX + lx + NG;
            }
            const int x = bc_cell(min(x0 + lx, g.n[0] + NG - 1), g.n[0], g.bc[0], g.bc[1]);
            const int y = bc_cell(min(y0 + ly, g.n[1] + NG - 1), g.n[1], g.bc[2], g.bc[3]);
            z = bc_cell(z, g.n[2], g.bc[4], g.bc[5]);
            const T *s = q + (int64_t)(z + NG) * g.stride[2] + (int64_t)(y + NG) * g.stride[1] + (x + NG);
#pragma unroll
            for (int v = 0; v < NV; v++) qc[j][v] = s[v * g.vstride];
        }
#pragma unroll
        for (int j = 0; j < 2; j++) {
            if (at[j] < 0 && col[j] < 0) continue;
            T w[NV];
            bad |= cons_to_prim<3, T>(g, qc[j], w);
#pragma unroll
            for (int v = 0; v < NV; v++) {
                if (at[j] >= 0) L.plane[v * PLANE + at[j]] = w[v];
                if (col[j] >= 0) L.column[v * NZ * NOWN + col[j]] = w[v];
            }
        }
    }
    __syncthreads();

    // ---- reconstruct: x cell col - 1 of row `row`; y row row - 1 of column
    // col; z plane k - 1 + m of cell `cell`
    const int sweep = t < Y0 ? 0 : (t < Z0 ? 1 : 2), p = t - (sweep == 0 ? 0 : (sweep == 1 ? Y0 : Z0));
    const bool rec = p < (sweep == 0 ? NPX : (sweep == 1 ? NPY : NPZ));
    const int width = sweep == 0 ? TX + 2 : (sweep == 1 ? TX : NOWN);
    const int row = p / width, col = p % width;   // z: m and the cell
    T wP[NV];
    if (rec) {
        const int step = sweep == 0 ? 1 : (sweep == 1 ? PX : NOWN);
        const T *st = sweep == 0 ? L.plane + (row + NG) * PX + col
                                 : (sweep == 1 ? L.plane + row * PX + col + NG : L.column + row * NOWN + col);
        const int vs = sweep == 2 ? NZ * NOWN : PLANE;
        st += (5 - ORDER) / 2 * step;   // WENO3 reads the inner three, first order the cell
#pragma unroll
        for (int v = 0; v < NV; v++) {
            const T *s = st + v * vs;
            T &m = L.minus[v * NT + t];
            if constexpr (ORDER == 5) weno5_pair(s[0], s[step], s[2 * step], s[3 * step], s[4 * step], T(g.eps), wP[v], m);
            else if constexpr (ORDER == 3) weno3_pair(s[0], s[step], s[2 * step], T(g.eps), wP[v], m);
            else wP[v] = m = s[0];
        }
    }
    __syncthreads();

    // ---- faces above the reconstructions; the operands of this thread's first
    // result are loaded ahead of them
    T a0[2], a1[2];
    auto operands = [&](int j) {
        const int r = t + j * NT, cell = r % NOWN, v = r / NOWN, x = x0 + cell % TX, y = y0 + cell / TX;
        if (r >= kResults || x >= g.n[0] || y >= g.n[1]) return;
        const int64_t c = v * g.vstride + (int64_t)(k + NG) * g.stride[2] + (int64_t)(y + NG) * g.stride[1] + (x + NG);
        a1[j] = q[c];
        a0[j] = mode == 1 ? a1[j] : q0[c];
    };
    operands(0);
    operands(1);
    {
        T wR[NV], F[NV], uf = T(0);
        const bool face = rec && (sweep == 0 ? col <= TX : (sweep == 1 ? row <= TY : row < 2));
        if (face) {
            const int up = t + (sweep == 0 ? 1 : width);
#pragma unroll
            for (int v = 0; v < NV; v++) wR[v] = L.minus[v * NT + up];
            bool b, counts;
            if (sweep == 0) {
                b = hllc<3, 0, T>(g, wP, wR, F, uf);
                counts = y0 + row < g.n[1] && x0 + col <= g.n[0];
            } else if (sweep == 1) {
                b = hllc<3, 1, T>(g, wP, wR, F, uf);
                counts = x0 + col < g.n[0] && y0 + row <= g.n[1];
            } else {
                b = hllc<3, 2, T>(g, wP, wR, F, uf);
                counts = x0 + col % TX < g.n[0] && y0 + col / TX < g.n[1];
            }
            bad |= b && counts;
#pragma unroll
            for (int v = 0; v < NV; v++) L.flux[v * NT + t] = F[v];
            L.flux[NV * NT + t] = uf;
        }
    }
    __syncthreads();

    // ---- results, one (cell, variable) after the other: the x+y part of the
    // stage combination and then the z part, as the split kernels form them
    double m = 0.0;
    if (ss.speeds)
        for (int w = 0; w < NT / 64; w++) m = __builtin_fmax(m, L.speed[w]);
    const T hdt = T(ss.finish(m, blockIdx.x == 0 && t == 0)), idx = T(g.inv_dx[0]), idy = T(g.inv_dx[1]), idz = T(g.inv_dx[2]);
    const T ca = T(mode == 2 ? 0.75 : (mode == 3 ? 1.0 / 3.0 : 0.0));
    const T cb = T(mode == 2 ? 0.25 : (mode == 3 ? 2.0 / 3.0 : 1.0));
#pragma unroll
    for (int j = 0; j < 2; j++) {
        const int r = t + j * NT, cell = r % NOWN, v = r / NOWN, tx = cell % TX, ty = cell / TX;
        const int x = x0 + tx, y = y0 + ty;
        if (r >= kResults || x >= g.n[0] || y >= g.n[1]) continue;
        const int fx = ty * (TX + 2) + tx, fy = Y0 + ty * TX + tx, fz = Z0 + cell;
        const T *F = L.flux + v * NT, *u = L.flux + NV * NT;
        T Lxy = (F[fx] - F[fx + 1]) * idx;
        Lxy += (F[fy] - F[fy + TX]) * idy;
        T Lz = (F[fz] - F[fz + NOWN]) * idz;
        if (v == A) {
            const int o = (ty + NG) * PX + tx + NG;
            const T h = alpha_source<T>(g, L.plane[A * PLANE + o], L.plane[E * PLANE + o]);
            T divu = (u[fx + 1] - u[fx]) * idx;
            divu += (u[fy + TX] - u[fy]) * idy;
            Lxy += h * divu;
            Lz += h * ((u[fz + NOWN] - u[fz]) * idz);
        }
        const T res = (mode == 1 ? a1[j] + hdt * Lxy : ca * a0[j] + cb * (a1[j] + hdt * Lxy)) + (cb * hdt) * Lz;
        out[v * g.vstride + (int64_t)(k + NG) * g.stride[2] + (int64_t)(y + NG) * g.stride[1] + (x + NG)] = res;
        L.minus[r] = res;   // last read before the third barrier
    }
    if (ss.carry) {   // wave speeds of the results (three wavefronts)
        static_assert(NOWN <= 192, "the cells of three wavefronts");
        __syncthreads();
        if (t < 192) {
            double sp = 0.0;
            if (t < NOWN && x0 + t % TX < g.n[0] && y0 + t / TX < g.n[1]) {
                T r[NV], w[NV];
#pragma unroll
                for (int v = 0; v < NV; v++) r[v] = L.minus[v * NOWN + t];
                cons_to_prim<3, T>(g, r, w);
                double Gam, Pi;
                mixture<double>(g, double(w[A]), Gam, Pi);
                const double cs = sqrtT(sound2<double>(Gam, Pi, double(w[0]) + double(w[1]), double(w[E])));
#pragma unroll
                for (int d = 0; d < 3; d++) sp = __builtin_fmax(sp, __builtin_fabs(double(w[2 + d])) + cs);
            }
            sp = wave_max(sp);
            if (t % 64 == 0) ss.carry[blockIdx.x * 3 + t / 64] = sp;
        }
    }
    if (bad) raise_flag(flag, 1);
}

int64_t tiles(const Grid &g)
{
    return (int64_t)((g.n[0] + TX - 1) / TX) * ((g.n[1] + TY - 1) / TY) * g.n[2];
}

template <class T, int ORDER>
int launch(mfc_grid *h, const void *q, const void *q0, void *out, int mode, const StepSize &ss, hipStream_t s)
{
    const Grid &g = h->g;
    hipLaunchKernelGGL((k_cube<T, ORDER>), dim3((unsigned)tiles(g)), dim3(NT), 0, s, g, (const T *)q, (const T *)q0, (T *)out,
                       mode, ss, (g.n[0] + TX - 1) / TX, (g.n[1] + TY - 1) / TY, h->flag);
    return hip_status(hipGetLastError(), "small 3D right-hand side launch");
}

template <class T>
int launch_t(mfc_grid *h, const void *q, const void *q0, void *out, int mode, const StepSize &ss, hipStream_t s)
{
    switch (h->desc.recon) {
    case MFC_RECON_WENO3: return launch<T, 3>(h, q, q0, out, mode, ss, s);
    case MFC_RECON_FIRST_ORDER: return launch<T, 1>(h, q, q0, out, mode, ss, s);
    default: return launch<T, 5>(h, q, q0, out, mode, ss, s);
    }
}

}  // namespace

// none where the grid is past any rule's reach
int64_t cube_partials(const Grid &g) { return tiles(g) <= 1024 ? 3 * tiles(g) : 0; }

// One workgroup per CU at most.  A step against the split kernels, FP64: 16^3
// (32 tiles) 51 -> 34 us, 24^3 (144) 52 -> 37, 32 x 30 x 32 (192) 55 -> 41; in
// two rounds 36 x 34 x 33 (396) 63 -> 65, 48^3 (720) 80 -> 98.  FP32: 47 -> 30,
// 48 -> 35, and 52 -> 55.  Non-uniform cells, characteristic faces and the
// routed reconstruction take the split kernels, as do the bare right-hand side
// (mfc_rhs_noalloc gives its bits) and the timing of single kernels, which
// counts theirs.
bool takes_cube(const mfc_grid *h)
{
    return h->desc.kernel == MFC_KERNEL_SPLIT && h->desc.recon != MFC_RECON_LEARNED && !h->g.stretched && !h->g.cbc_mask &&
           !h->timing && tiles(h->g) <= std::min(h->cu_count, 1024);
}

int launch_rhs_cube(mfc_grid *h, const void *q, const void *q0, void *out, int mode, const StepSize &ss, hipStream_t s)
{
    return h->desc.precision == MFC_FP32_MIXED ? launch_t<float>(h, q, q0, out, mode, ss, s)
                                               : launch_t<double>(h, q, q0, out, mode, ss, s);
}

}  // namespace mfc
