// 2D right-hand side of a single grid (MFC_KERNEL_FUSED): one workgroup per
// tile of tile2.h, one launch per Runge-Kutta stage.
//
// A step is its three stage launches: neighbours past a face are read through
// the boundary rule, so no ghost fill runs before a stage; the last stage of
// a step followed by another of the same run reduces the wave speeds of the
// state it writes, from which the next step's first stage sets the step size.  A bare right-hand side (mode 0) reads the caller's ghost
// cells.
#include <cmath>

#include "tile2.h"

namespace mfc {
namespace {

// 16 x 14 cells: 252 and 256 reconstructions for the 256 threads of a sweep.
// FP64 (74 KB of LDS) fits two workgroups per CU, FP32 (37 KB) four.
using S2 = Tile2<16, 14>;

template <class T, bool ROUTE>
constexpr int kPlaneWaves = ROUTE ? 2 : 4;   // wavefronts per SIMD

template <class T, bool ROUTE, int ORDER, bool STRETCH>
__global__ void __launch_bounds__(S2::NT, (kPlaneWaves<T, ROUTE>))
    k_plane(Grid g, const T *__restrict__ q, const T *q0, T *out, int mode, StepSize ss, int tiles_x,
            int *__restrict__ flag, const float *__restrict__ mlpw, float logit_tau, T sqrt_eps)
{
    __shared__ Tile2Lds<T, S2> L;
    __shared__ __align__(16) typename std::conditional<ROUTE, mlp::Params, char>::type s_mlp;
    __shared__ __align__(16) uint16_t s_feat[ROUTE ? S2::NT * 16 : 1];
    const Role2<S2> R;
    const int x0 = (int)(blockIdx.x % tiles_x) * S2::TX, y0 = (int)(blockIdx.x / tiles_x) * S2::TY;
    T qc[6];
    bool read = false, bad = false;
    if (R.loads) read = load_cell2<T>(g, q, x0 + R.lx, y0 + R.ly, mode != 0, inner2<S2>(g, x0, y0), qc);
    const mlp::Params *net = nullptr;
    if constexpr (ROUTE) {   // visible after the tile's first barrier
        mlp::stage_params(s_mlp, nullptr, mlpw, threadIdx.x, S2::NT, true);
        net = &s_mlp;
    }
    const bool speed = ss.carry != nullptr;
    __shared__ double s_speed[S2::NT / 64];   // gathered by the tile's first barrier
    if (ss.speeds) {
        const double m = ss.gather(S2::NT);
        if (threadIdx.x % 64 == 0) s_speed[threadIdx.x / 64] = m;
    }
    auto step_size = [&] {
        double m = 0.0;
        if (ss.speeds)
#pragma unroll
            for (int w = 0; w < S2::NT / 64; w++) m = __builtin_fmax(m, s_speed[w]);
        return ss.finish(m, blockIdx.x == 0 && threadIdx.x == 0);
    };
    const double sp = tile2_stage<T, S2, ROUTE, ORDER, STRETCH, false>(
        g, L, R, x0, y0, qc, read, q, q0, out, mode, speed, bad, net, s_feat + (ROUTE ? threadIdx.x / 64 * 64 * 16 : 0),
        logit_tau, sqrt_eps, [] {}, step_size);
    if (speed && R.sweep == 0) {
        const double m = wave_max(sp);
        if (threadIdx.x % 64 == 0) ss.carry[blockIdx.x * (S2::NS / 64) + threadIdx.x / 64] = m;
    }
    if (bad) raise_flag(flag, 1);
}

template <class T, bool ROUTE, int ORDER, bool STRETCH>
int rhs_plane(mfc_grid *h, const void *q, const void *q0, void *out, int mode, const StepSize &ss, hipStream_t s)
{
    const Grid &g = h->g;
    const int tiles_x = (g.n[0] + S2::TX - 1) / S2::TX;
    const int64_t tiles = (int64_t)tiles_x * ((g.n[1] + S2::TY - 1) / S2::TY);
    timing_begin(h, s);
    hipLaunchKernelGGL((k_plane<T, ROUTE, ORDER, STRETCH>), dim3((unsigned)tiles), dim3(S2::NT), 0, s, g, (const T *)q,
                       (const T *)q0, (T *)out, mode, ss, tiles_x, h->flag, h->mlp, h->logit_tau,
                       T(__builtin_sqrt(g.weno_eps)));
    timing_end(h, s);
    return hip_status(hipGetLastError(), "2D right-hand side launch");
}

template <class T>
int rhs_plane_t(mfc_grid *h, const void *q, const void *q0, void *out, int mode, const StepSize &ss, hipStream_t s)
{
    const int recon = h->desc.recon;
    if (h->g.stretched)   // WENO5 or first order (validated at init)
        return recon == MFC_RECON_FIRST_ORDER ? rhs_plane<T, false, 1, true>(h, q, q0, out, mode, ss, s)
                                              : rhs_plane<T, false, 5, true>(h, q, q0, out, mode, ss, s);
    switch (recon) {
    case MFC_RECON_LEARNED: return rhs_plane<T, true, 5, false>(h, q, q0, out, mode, ss, s);
    case MFC_RECON_WENO3: return rhs_plane<T, false, 3, false>(h, q, q0, out, mode, ss, s);
    case MFC_RECON_FIRST_ORDER: return rhs_plane<T, false, 1, false>(h, q, q0, out, mode, ss, s);
    default: return rhs_plane<T, false, 5, false>(h, q, q0, out, mode, ss, s);
    }
}

}  // namespace

int64_t plane_partials(const Grid &g)
{
    return (int64_t)((g.n[0] + S2::TX - 1) / S2::TX) * ((g.n[1] + S2::TY - 1) / S2::TY) * (S2::NS / 64);
}

int launch_rhs_plane(mfc_grid *h, const void *q, const void *q0, void *out, int mode, const StepSize &ss, hipStream_t s)
{
    if (h->desc.recon == MFC_RECON_LEARNED && !h->mlp)
        return fail(MFC_E_ARG, "MFC_RECON_LEARNED needs mfc_set_indicator first");
    return h->desc.precision == MFC_FP32_MIXED ? rhs_plane_t<float>(h, q, q0, out, mode, ss, s)
                                               : rhs_plane_t<double>(h, q, q0, out, mode, ss, s);
}

}  // namespace mfc
