// Learned smoothness indicator (project extension beside Sec. 3.2): harvest
// of training samples from a solver state, training of the perceptron of
// mlp.h with the project's own bf16 matrix-core forward and backward kernels
// (FP32 master weights, mean binary cross-entropy, Adam), batched inference,
// and the handle call that installs a trained network for the routed
// reconstruction.
//
//   k_harvest     one thread per interior cell, every direction: the 15 inputs
//                 and the label "every variable keeps its WENO5 weights
//                 within 0.01 of the ideal ones on both faces";
//   k_mlp_grad    forward + backward over a batch; each wavefront walks
//                 16-sample tiles, keeps the weight-gradient tiles in MFMA
//                 accumulators and the bias/W3 gradients in registers; a
//                 workgroup writes one partial sum of all 1601 gradients and
//                 the loss;
//   k_mlp_reduce  sums the partials in a fixed order (deterministic);
//   k_adam        one thread per parameter;
//   k_mlp_infer   P(smooth) of a list of samples.
#include <cmath>
#include <new>

#include "internal.h"
#include "mlp.h"

struct mfc_trainer {
    int64_t max_batch = 0;
    int blocks = 0;
    int device = 0;
    float *w = nullptr, *m = nullptr, *v = nullptr;  // master weights, Adam moments
    float *grad = nullptr;                           // [NPARAM + 1]: gradients, loss
    float *partial = nullptr;                        // [blocks][NPARAM + 1]
    int64_t step = 0;                                // Adam steps taken
    bool have_grad = false;
};

namespace mfc {
namespace {

using namespace mlp;
constexpr int kThreads = 256, kWaves = kThreads / 64;
constexpr int NP1 = NPARAM + 1;

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Largest |omega_r - d_r| of WENO5-JS over the three stencils and both faces
// of the 5-cell stencil v (the weights of Sec. 3.2).  As in the solver's
// weno5_pair, e_r = 3/4 (eps + beta_r) in the divided differences of the
// stencil and omega_r through common denominators (omega_0 ~ 1 (e_1 e_2)^2
// and so on, ideal weights times ten), which leaves one reciprocal per face;
// these are refined to the last place.  The denominators are fourth powers
// of e_r; where they leave the normal numbers (differences above 1e38, or below
// 1e-38 with an epsilon to match), `rare` is set and the caller takes the
// weights as they are defined instead (BY_SQUARES).
template <bool BY_SQUARES = false>
__device__ __forceinline__ double weno_deviation(const double *v, double eps, bool &rare)
{
    const double b = v[1] - v[0], a = v[2] - v[1], c = v[3] - v[2], d = v[4] - v[3];
    const double e3 = 0.75 * eps;
    const double e0 = __builtin_fma(a, __builtin_fma(2.5, a, -2.75 * b), __builtin_fma(b, b, e3));
    const double e1 = __builtin_fma(c, __builtin_fma(-1.25, a, c), __builtin_fma(a, a, e3));
    const double e2 = __builtin_fma(c, __builtin_fma(2.5, c, -2.75 * d), __builtin_fma(d, d, e3));
    const double s0 = e0 * e0, s1 = e1 * e1, s2 = e2 * e2;
    if constexpr (BY_SQUARES) {
        const double s[3] = {s0, s1, s2}, d[3] = {0.1, 0.6, 0.3};
        double ap[3], am[3], dev = 0.0;
#pragma unroll
        for (int r = 0; r < 3; r++) {
            ap[r] = d[r] / s[r];
            am[r] = d[2 - r] / s[r];
        }
        const double sp = ap[0] + ap[1] + ap[2], sm = am[0] + am[1] + am[2];
#pragma unroll
        for (int r = 0; r < 3; r++) dev = fmax(dev, fmax(fabs(ap[r] / sp - d[r]), fabs(am[r] / sm - d[2 - r])));
        return dev;
    }
    const double m0 = s1 * s2, m1 = 6.0 * (s0 * s2), m2 = s0 * s1;
    const double sp = __builtin_fma(3.0, m2, m0 + m1);   // + face: weights 1, 6, 3
    const double sm = __builtin_fma(3.0, m0, m1 + m2);   // - face: weights 3, 6, 1
    rare |= !normal(sp) || !normal(sm);
    const double rp = divisor(sp), rm = divisor(sm);
    double dev = fmax(fabs(__builtin_fma(m0, rp, -0.1)), fabs(__builtin_fma(m1, rp, -0.6)));
    dev = fmax(dev, fabs(__builtin_fma(3.0 * m2, rp, -0.3)));
    dev = fmax(dev, fabs(__builtin_fma(3.0 * m0, rm, -0.3)));
    dev = fmax(dev, fabs(__builtin_fma(m1, rm, -0.6)));
    return fmax(dev, fabs(__builtin_fma(m2, rm, -0.1)));
}

// Harvest tile: 256 cells, one per thread, which forms its cell's samples of
// every direction.  The tile's primitives with their halos of two cells are
// converted once into LDS (3D: 768 conversions for 768 samples instead of
// five per sample); the pressure as the two factors of its product.  Bound by the FP64 issue of the deviations.
template <int NDIM>
struct HarvestTile {
    static constexpr int H = 2, NV = 4 + NDIM;
    static constexpr int TX = NDIM == 1 ? 256 : (NDIM == 2 ? 16 : 8), TY = NDIM == 1 ? 1 : (NDIM == 2 ? 16 : 8);
    static constexpr int TZ = NDIM == 3 ? 4 : 1;
    static constexpr int OY = NDIM >= 2 ? H : 0, OZ = NDIM == 3 ? H : 0;   // halo depth in y and z
    // positions: the tile's cells, then the halo cells of its x, y and z faces
    // (no edges or corners: three 49 KB workgroups per CU in 3D)
    static constexpr int HX = 2 * H * TY * TZ, HY = 2 * OY * TX * TZ, HZ = 2 * OZ * TX * TY;
    static constexpr int CELLS = TX * TY * TZ, N = CELLS + HX + HY + HZ;
    static __device__ __forceinline__ int at(int x, int y, int z)
    {
        if (x < 0 || x >= TX) return CELLS + (z * TY + y) * 2 * H + (x < 0 ? x + H : x - TX + H);
        if (y < 0 || y >= TY) return CELLS + HX + (z * 2 * H + (y < 0 ? y + H : y - TY + H)) * TX + x;
        if (z < 0 || z >= TZ) return CELLS + HX + HY + ((z < 0 ? z + H : z - TZ + H) * TY + y) * TX + x;
        return (z * TY + y) * TX + x;
    }
    static_assert(TX * TY * TZ == kThreads, "one cell per thread");
};

// 96^3 cells: 192 us with one thread per (cell, direction), five conversions
// and 99 IEEE divisions per sample; 86 us so (14 reciprocals).
template <int NDIM>
__global__ void __launch_bounds__(kThreads, 3)
    k_harvest(Grid g, const double *__restrict__ q, uint16_t *__restrict__ X, uint8_t *__restrict__ Y,
              double *__restrict__ D, double sqrt_eps, double threshold, int64_t cells)
{
    using S = HarvestTile<NDIM>;
    constexpr int NV = S::NV, H = S::H;
    constexpr int E = NV - 2, A = NV - 1;
    __shared__ double s_w[NV][S::N];   // row E: the pressure's first factor
    __shared__ double s_ig[S::N];      // its second
    const int tid = threadIdx.x;
    const int tx = tid % S::TX, ty = (tid / S::TX) % S::TY, tz = tid / (S::TX * S::TY);
    const int tiles_x = (g.n[0] + S::TX - 1) / S::TX, tiles_y = (g.n[1] + S::TY - 1) / S::TY;
    const int x0 = blockIdx.x % tiles_x * S::TX, y0 = blockIdx.x / tiles_x % tiles_y * S::TY;
    const int z0 = blockIdx.x / tiles_x / tiles_y * S::TZ;
    // position (i, j, k) of the tile's window, from its first interior cell;
    // those past a ragged tile's last halo load a duplicate that no sample of the grid reads
    auto stage = [&](int i, int j, int k) {
        const int x = min(x0 + i, g.n[0] + H - 1), y = min(y0 + j, g.n[1] - 1 + S::OY), z = min(z0 + k, g.n[2] - 1 + S::OZ);
        const int64_t o = (int64_t)(z + g.off[2]) * g.stride[2] + (int64_t)(y + g.off[1]) * g.stride[1] + (x + g.off[0]);
        double qc[NV], w[NV], pf[2];
#pragma unroll
        for (int v = 0; v < NV; v++) qc[v] = q[v * g.vstride + o];
        (void)cons_to_prim<NDIM, double>(g, qc, w, pf);
        w[E] = pf[0];
        const int p = S::at(i, j, k);
#pragma unroll
        for (int v = 0; v < NV; v++) s_w[v][p] = w[v];
        s_ig[p] = pf[1];
    };
    stage(tx, ty, tz);
    for (int h = tid; h < S::HX + S::HY + S::HZ; h += kThreads) {
        int a, i, j, k;
        if (h < S::HX) {
            a = h % (2 * H);
            j = (h / (2 * H)) % S::TY;
            k = h / (2 * H * S::TY);
            i = a < H ? a - H : S::TX + a - H;
        } else if (h < S::HX + S::HY) {
            const int r = h - S::HX;
            i = r % S::TX;
            a = (r / S::TX) % (2 * H);
            k = r / (S::TX * 2 * H);
            j = a < H ? a - H : S::TY + a - H;
        } else {
            const int r = h - S::HX - S::HY;
            i = r % S::TX;
            j = (r / S::TX) % S::TY;
            a = r / (S::TX * S::TY);
            k = a < H ? a - H : S::TZ + a - H;
        }
        stage(i, j, k);
    }
    __syncthreads();
    const int x = x0 + tx, y = y0 + ty, z = z0 + tz;
    if (x >= g.n[0] || y >= g.n[1] || z >= g.n[2]) return;
    const int64_t c = ((int64_t)z * g.n[1] + y) * g.n[0] + x;
    const int p = tid;
    const int d0 = gridDim.y > 1 ? (int)blockIdx.y : 0, d1 = gridDim.y > 1 ? d0 + 1 : NDIM;   // one direction, or all
#pragma unroll 1
    for (int d = d0; d < d1; d++) {
        const int64_t t = d * cells + c;
        int at[5];   // the stencil's positions
#pragma unroll
        for (int j = 0; j < 5; j++) at[j] = S::at(tx + (d == 0 ? j - 2 : 0), ty + (d == 1 ? j - 2 : 0), tz + (d == 2 ? j - 2 : 0));
        // Differences to the centre.  The pressure's are taken before the
        // rounding of the neighbour's product (one FMA), except the one next
        // above the centre: where pressures differ by rounding alone these
        // set the features' bits, and samples keep their bits.  The weights
        // are those of the rounded values.
        double dif[3][5], pr[5];
        const double a2 = s_w[A][p], r2 = s_w[0][p] + s_w[1][p];
        double pr2 = s_w[E][p] * s_ig[p];
        __asm__("" : "+v"(pr2));   // rounded
#pragma unroll
        for (int j = 0; j < 5; j++) {
            const int o = at[j];
            dif[0][j] = s_w[A][o] - a2;
            dif[1][j] = (s_w[0][o] + s_w[1][o]) - r2;
            pr[j] = s_w[E][o] * s_ig[o];
            __asm__("" : "+v"(pr[j]));   // rounded
            dif[2][j] = j == 3 ? pr[j] - pr2 : __builtin_fma(s_w[E][o], s_ig[o], -pr2);
        }
        uint16_t f[16];
        features_of<double>(dif, sqrt_eps, f);
        uint4 *xo = (uint4 *)(X + t * 16);
        const uint32_t *f32 = (const uint32_t *)f;
        xo[0] = make_uint4(f32[0], f32[1], f32[2], f32[3]);
        xo[1] = make_uint4(f32[4], f32[5], f32[6], f32[7]);
        double dev = 0.0;
        bool rare = false;
#pragma unroll
        for (int v = 0; v < NV; v++) {
            double st[5];
#pragma unroll
            for (int j = 0; j < 5; j++) st[j] = v == E ? pr[j] : s_w[v][at[j]];
            dev = fmax(dev, weno_deviation(st, g.weno_eps, rare));
        }
        if (__builtin_expect(rare, 0)) {
            dev = 0.0;
#pragma unroll 1
            for (int v = 0; v < NV; v++) {
                double st[5];
#pragma unroll
                for (int j = 0; j < 5; j++) st[j] = v == E ? pr[j] : s_w[v][at[j]];
                dev = fmax(dev, weno_deviation<true>(st, g.weno_eps, rare));
            }
        }
        Y[t] = dev < threshold ? 1 : 0;
        if (D) D[t] = dev;
    }
}

__global__ void __launch_bounds__(kThreads)
    k_mlp_grad(const float *__restrict__ w, const uint16_t *__restrict__ X, const uint8_t *__restrict__ Y,
               const int *__restrict__ index, int64_t batch, float inv_n, float *__restrict__ partial)
{
    __shared__ __align__(16) Params P;
    __shared__ __align__(16) ParamsT PT;
    __shared__ __align__(16) uint16_t sx[kWaves][16 * 16];   // X tile [sample][feature]
    __shared__ __align__(16) uint16_t sh1[kWaves][16 * NH];  // H1 tile [sample][unit]
    __shared__ __align__(16) uint16_t sd2[kWaves][16 * NH];  // dZ2 tile
    __shared__ __align__(16) uint16_t sd1[kWaves][16 * NH];  // dZ1 tile
    __shared__ float red[kWaves][NP1];
    const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64, g = lane >> 4, s = lane & 15;
    // the operands of a tile are loaded ahead (the first tile's with the
    // parameters): an index, then the features and label it names
    const int64_t ntiles = (batch + 15) / 16, stride = (int64_t)gridDim.x * kWaves;
    int64_t tile = (int64_t)blockIdx.x * kWaves + wave;
    s4 xn = s4{0, 0, 0, 0};
    float yn = 0.f;
    auto fetch = [&](int64_t t) {
        const int64_t smp = t * 16 + s;
        const bool valid = smp < batch;
        const int64_t row = valid ? (index ? (int64_t)index[smp] : smp) : 0;
        xn = valid ? *(const s4 *)(X + row * 16 + 4 * g) : s4{0, 0, 0, 0};
        yn = valid ? float(Y[row]) : 0.f;
    };
    if (tile < ntiles) fetch(tile);
    stage_params(P, &PT, w, tid, kThreads);
    __syncthreads();

    f4 aw1[2], aw2[2][2];
#pragma unroll
    for (int b = 0; b < 2; b++) {
        aw1[b] = f4{0.f, 0.f, 0.f, 0.f};
        aw2[b][0] = aw2[b][1] = f4{0.f, 0.f, 0.f, 0.f};
    }
    float dw3[8], db2[8], db1[8], db3 = 0.f, loss = 0.f;
#pragma unroll
    for (int q = 0; q < 8; q++) dw3[q] = db2[q] = db1[q] = 0.f;

    for (; tile < ntiles; tile += stride) {
        const bool valid = tile * 16 + s < batch;
        const s4 xb = xn;
        const float y = yn;
        if (tile + stride < ntiles) fetch(tile + stride);
        Fwd F;
        forward_tile(P, xb, lane, F);
        const float prob = 1.0f / (1.0f + __expf(-F.z));
        const float dz = valid ? (prob - y) * inv_n : 0.f;
        if (g == 0) {
            db3 += dz;
            if (valid) loss += fmaxf(F.z, 0.f) - F.z * y + log1pf(__expf(-fabsf(F.z)));
        }
        float dz2[8];
        uint16_t dz2_bits[8];
        bf8 dz2b;
#pragma unroll
        for (int q = 0; q < 8; q++) {
            const int u = 16 * (q / 4) + 4 * g + (q % 4);
            dw3[q] += dz * F.h2[q];
            dz2[q] = P.w3[u] * dz * gelu_grad(F.z2[q]);
            db2[q] += dz2[q];
            dz2_bits[q] = bf16_bits(dz2[q]);
            dz2b[q] = as_bf16(dz2_bits[q]);
        }
        float dz1[8];
#pragma unroll
        for (int b = 0; b < 2; b++) {
            f4 c = f4{0.f, 0.f, 0.f, 0.f};
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(PT.a2t[b][lane], dz2b, c, 0, 0, 0);
#pragma unroll
            for (int t = 0; t < 4; t++) {
                dz1[4 * b + t] = c[t] * gelu_grad(F.z1[4 * b + t]);
                db1[4 * b + t] += dz1[4 * b + t];
            }
        }
        // stage the tiles [sample][unit] for the sample-contracted products
        *(s4 *)&sx[wave][s * 16 + 4 * g] = xb;
#pragma unroll
        for (int q = 0; q < 8; q++) {
            const int u = unit(g, q);
            sh1[wave][s * NH + u] = F.h1_bits[q];
            sd2[wave][s * NH + u] = dz2_bits[q];
            sd1[wave][s * NH + u] = bf16_bits(dz1[q]);
        }
        wave_sync();
        // dW1 [16 f x 32 u] += X^T dZ1, dW2 [32 in x 32 out] += H1^T dZ2 (k = samples)
        s4 ax;
#pragma unroll
        for (int t = 0; t < 4; t++) ax[t] = (short)sx[wave][(4 * g + t) * 16 + s];
#pragma unroll
        for (int bu = 0; bu < 2; bu++) {
            s4 bz;
#pragma unroll
            for (int t = 0; t < 4; t++) bz[t] = (short)sd1[wave][(4 * g + t) * NH + 16 * bu + s];
            aw1[bu] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ax, bz, aw1[bu], 0, 0, 0);
        }
#pragma unroll
        for (int bi = 0; bi < 2; bi++) {
            s4 ah;
#pragma unroll
            for (int t = 0; t < 4; t++) ah[t] = (short)sh1[wave][(4 * g + t) * NH + 16 * bi + s];
#pragma unroll
            for (int bo = 0; bo < 2; bo++) {
                s4 bz;
#pragma unroll
                for (int t = 0; t < 4; t++) bz[t] = (short)sd2[wave][(4 * g + t) * NH + 16 * bo + s];
                aw2[bi][bo] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ah, bz, aw2[bi][bo], 0, 0, 0);
            }
        }
        wave_sync();
    }

    // wavefront partials -> red[wave][flat index]
    float *r = red[wave];
#pragma unroll
    for (int b = 0; b < 2; b++)
#pragma unroll
        for (int t = 0; t < 4; t++) {
            const int f = 4 * g + t;
            if (f < NIN) r[OW1 + f * NH + 16 * b + s] = aw1[b][t];
#pragma unroll
            for (int bo = 0; bo < 2; bo++) r[OW2 + (16 * b + 4 * g + t) * NH + 16 * bo + s] = aw2[b][bo][t];
        }
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
#pragma unroll
        for (int q = 0; q < 8; q++) {
            dw3[q] += __shfl_xor(dw3[q], o, 64);
            db2[q] += __shfl_xor(db2[q], o, 64);
            db1[q] += __shfl_xor(db1[q], o, 64);
        }
        db3 += __shfl_xor(db3, o, 64);
        loss += __shfl_xor(loss, o, 64);
    }
    if (s == 0) {
#pragma unroll
        for (int q = 0; q < 8; q++) {
            const int u = 16 * (q / 4) + 4 * g + (q % 4);
            r[OW3 + u] = dw3[q];
            r[OB2 + u] = db2[q];
            r[OB1 + u] = db1[q];
        }
        if (g == 0) {
            r[OB3] = db3;
            r[NPARAM] = loss;
        }
    }
    __syncthreads();
    for (int e = tid; e < NP1; e += kThreads)
        partial[(int64_t)blockIdx.x * NP1 + e] = (red[0][e] + red[1][e]) + (red[2][e] + red[3][e]);
}

// Sums the workgroup partials of every gradient in workgroup order (a fixed
// order: deterministic).  The launch is the latency of its loads: a workgroup
// owns 64 gradients (26 workgroups) and its 16 wavefronts load 64 rows of
// partials at once, the next 64 while the first wavefront adds this lot from
// LDS.  64 partials (a batch of 4096): 16.0 us with one thread per gradient
// loading row after row, 2.8 us so.
constexpr int kRedE = 64, kRedWaves = 16, kRedRows = 64, kRedPer = kRedRows / kRedWaves;
__global__ void __launch_bounds__(64 * kRedWaves)
    k_mlp_reduce(const float *__restrict__ partial, int blocks, float *__restrict__ out, float inv_n)
{
    __shared__ float rows[kRedRows][kRedE];
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64, e = blockIdx.x * kRedE + lane;
    const int ec = e < NP1 ? e : NP1 - 1;   // lanes past the end load a duplicate
    float next[kRedPer], acc = 0.f;
    auto fetch = [&](int b0) {
#pragma unroll
        for (int j = 0; j < kRedPer; j++) {
            const int b = b0 + wave * kRedPer + j;
            next[j] = b < blocks ? partial[(int64_t)b * NP1 + ec] : 0.f;
        }
    };
    fetch(0);
    for (int b0 = 0; b0 < blocks; b0 += kRedRows) {
#pragma unroll
        for (int j = 0; j < kRedPer; j++) rows[wave * kRedPer + j][lane] = next[j];
        __syncthreads();
        if (b0 + kRedRows < blocks) fetch(b0 + kRedRows);
        if (wave == 0) {
            const int n = blocks - b0 < kRedRows ? blocks - b0 : kRedRows;
#pragma unroll 16
            for (int j = 0; j < n; j++) acc += rows[j][lane];
        }
        __syncthreads();
    }
    if (wave == 0 && e < NP1) out[e] = e == NPARAM ? acc * inv_n : acc;   // the loss is a mean
}

__global__ void k_adam(float *__restrict__ w, float *__restrict__ m, float *__restrict__ v,
                       const float *__restrict__ grad, float lr, float b1, float b2, float c1, float c2, float eps)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= NPARAM) return;
    const float gr = grad[e];
    const float mm = b1 * m[e] + (1.0f - b1) * gr;
    const float vv = b2 * v[e] + (1.0f - b2) * gr * gr;
    m[e] = mm;
    v[e] = vv;
    w[e] -= lr * (mm / c1) / (sqrtf(vv / c2) + eps);
}

__global__ void __launch_bounds__(kThreads)
    k_mlp_infer(const float *__restrict__ w, const uint16_t *__restrict__ X, int64_t n, float *__restrict__ prob)
{
    __shared__ __align__(16) Params P;
    const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64, g = lane >> 4, s = lane & 15;
    stage_params(P, nullptr, w, tid, kThreads);
    __syncthreads();
    const int64_t ntiles = (n + 15) / 16;
    for (int64_t tile = (int64_t)blockIdx.x * kWaves + wave; tile < ntiles; tile += (int64_t)gridDim.x * kWaves) {
        const int64_t smp = tile * 16 + s;
        s4 xb = smp < n ? *(const s4 *)(X + smp * 16 + 4 * g) : s4{0, 0, 0, 0};
        const float z = logit_tile(P, xb, lane);
        if (g == 0 && smp < n) prob[smp] = 1.0f / (1.0f + __expf(-z));
    }
}

// The logit of all-zero features behind a routed network's parameters, by the
// same tile products as any sample's.
__global__ void __launch_bounds__(kThreads) k_zero_logit(float *w)
{
    __shared__ __align__(16) Params P;
    stage_params(P, nullptr, w, threadIdx.x, kThreads);
    __syncthreads();
    const float z = logit_tile(P, s4{0, 0, 0, 0}, threadIdx.x % 64);
    if (threadIdx.x == 0) w[NPARAM] = z;
}

}  // namespace
}  // namespace mfc

using namespace mfc;

extern "C" {

int mfc_harvest(mfc_grid *h, void *q, uint16_t *features, uint8_t *labels, double *maxdev, void *stream)
{
    if (!h || !q || !features || !labels) return fail(MFC_E_ARG, "null argument");
    if (h->desc.precision != MFC_FP64) return fail(MFC_E_UNSUPPORTED, "harvest reads FP64 states");
    if (h->g.stretched) return fail(MFC_E_UNSUPPORTED, "harvest labels uniform-grid WENO5 weights");
    int st = mfc_fill_ghosts(h, q, stream);
    if (st) return st;
    hipStream_t s = (hipStream_t)stream;
    const double se = std::sqrt(h->g.weno_eps), *qd = (const double *)q;
    auto launch = [&](auto nd) {
        using S = HarvestTile<decltype(nd)::value>;
        const Grid &g = h->g;
        const int64_t tiles = (int64_t)((g.n[0] + S::TX - 1) / S::TX) * ((g.n[1] + S::TY - 1) / S::TY) *
                              ((g.n[2] + S::TZ - 1) / S::TZ);
        // few tiles: a workgroup per direction (their conversions formed again),
        // where one would walk them one after the other on an idle chip (8^3
        // cells with the ghost fill 20.1 -> 16.8 us, 24^3 21.2 -> 18.0)
        const unsigned split = tiles * decltype(nd)::value <= h->cu_count ? decltype(nd)::value : 1;
        hipLaunchKernelGGL(k_harvest<decltype(nd)::value>, dim3((unsigned)tiles, split), dim3(kThreads), 0, s, g, qd, features,
                           labels, maxdev, se, 0.01, h->cells);
    };
    if (h->g.ndim == 1) launch(std::integral_constant<int, 1>{});
    else if (h->g.ndim == 2) launch(std::integral_constant<int, 2>{});
    else launch(std::integral_constant<int, 3>{});
    return hip_status(hipGetLastError(), "harvest launch");
}

int mfc_trainer_free(mfc_trainer *t)
{
    if (!t) return MFC_OK;
    (void)hipDeviceSynchronize();
    for (void *p : {(void *)t->w, (void *)t->m, (void *)t->v, (void *)t->grad, (void *)t->partial})
        if (p) (void)hipFree(p);
    delete t;
    return MFC_OK;
}

int mfc_trainer_init(int64_t max_batch, mfc_trainer **out)
{
    if (!out) return fail(MFC_E_ARG, "out is NULL");
    *out = nullptr;
    if (max_batch < 1 || max_batch > (int64_t(1) << 31)) return fail(MFC_E_ARG, "max_batch must be in [1, 2^31]");
    mfc_trainer *t = new (std::nothrow) mfc_trainer();
    if (!t) return fail(MFC_E_NOMEM, "host allocation failed");
    t->max_batch = max_batch;
    int cu = 0;
    if (hipGetDevice(&t->device) != hipSuccess ||
        hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, t->device) != hipSuccess || cu <= 0) {
        delete t;
        return fail(MFC_E_HIP, "device query failed");
    }
    const int64_t tiles = (max_batch + 15) / 16;
    t->blocks = (int)std::min<int64_t>((tiles + kWaves - 1) / kWaves, (int64_t)2 * cu);
    hipError_t e = hipSuccess;
    auto alloc = [&](float **p, size_t n) {
        if (e == hipSuccess) e = hipMalloc((void **)p, n * sizeof(float));
    };
    alloc(&t->w, NPARAM);
    alloc(&t->m, NPARAM);
    alloc(&t->v, NPARAM);
    alloc(&t->grad, NP1);
    alloc(&t->partial, (size_t)t->blocks * NP1);
    if (e == hipSuccess) e = hipMemset(t->w, 0, NPARAM * sizeof(float));
    if (e == hipSuccess) e = hipMemset(t->m, 0, NPARAM * sizeof(float));
    if (e == hipSuccess) e = hipMemset(t->v, 0, NPARAM * sizeof(float));
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) {
        mfc_trainer_free(t);
        return fail(MFC_E_NOMEM, "trainer allocation failed");
    }
    *out = t;
    return MFC_OK;
}

int mfc_trainer_set_params(mfc_trainer *t, const float *params_host)
{
    if (!t || !params_host) return fail(MFC_E_ARG, "null argument");
    hipError_t e = hipMemcpy(t->w, params_host, NPARAM * sizeof(float), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemset(t->m, 0, NPARAM * sizeof(float));
    if (e == hipSuccess) e = hipMemset(t->v, 0, NPARAM * sizeof(float));
    if (e == hipSuccess) e = hipDeviceSynchronize();
    t->step = 0;
    t->have_grad = false;
    return hip_status(e, "trainer parameter upload");
}

int mfc_trainer_get_params(mfc_trainer *t, float *params_host)
{
    if (!t || !params_host) return fail(MFC_E_ARG, "null argument");
    return hip_status(hipMemcpy(params_host, t->w, NPARAM * sizeof(float), hipMemcpyDeviceToHost),
                      "trainer parameter download");
}

int mfc_trainer_grad(mfc_trainer *t, const uint16_t *features, const uint8_t *labels, const int32_t *index,
                     int64_t batch, void *stream)
{
    if (!t || !features || !labels) return fail(MFC_E_ARG, "null argument");
    if (batch < 1 || batch > t->max_batch) return fail(MFC_E_ARG, "batch must be in [1, max_batch]");
    hipStream_t s = (hipStream_t)stream;
    const float inv_n = (float)(1.0 / (double)batch);
    hipLaunchKernelGGL(k_mlp_grad, dim3(t->blocks), dim3(kThreads), 0, s, t->w, features, labels, index, batch, inv_n,
                       t->partial);
    hipLaunchKernelGGL(k_mlp_reduce, dim3((NP1 + kRedE - 1) / kRedE), dim3(64 * kRedWaves), 0, s, t->partial, t->blocks,
                       t->grad, inv_n);
    t->have_grad = true;
    return hip_status(hipGetLastError(), "gradient launch");
}

int mfc_trainer_read_grad(mfc_trainer *t, float *grad_host, float *loss_host, void *stream)
{
    if (!t || !grad_host) return fail(MFC_E_ARG, "null argument");
    if (!t->have_grad) return fail(MFC_E_ARG, "no gradient computed yet");
    float buf[NP1];
    hipStream_t s = (hipStream_t)stream;
    hipError_t e = hipMemcpyAsync(buf, t->grad, sizeof(buf), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_status(e, "gradient download");
    for (int i = 0; i < NPARAM; i++) grad_host[i] = buf[i];
    if (loss_host) *loss_host = buf[NPARAM];
    return MFC_OK;
}

int mfc_trainer_adam(mfc_trainer *t, float lr, float beta1, float beta2, float eps, void *stream)
{
    if (!t) return fail(MFC_E_ARG, "null argument");
    if (!t->have_grad) return fail(MFC_E_ARG, "no gradient computed yet");
    if (!(lr > 0.f) || !(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f) || !(eps > 0.f))
        return fail(MFC_E_ARG, "bad Adam hyper-parameters");
    t->step++;
    const float c1 = (float)(1.0 - std::pow((double)beta1, (double)t->step));
    const float c2 = (float)(1.0 - std::pow((double)beta2, (double)t->step));
    hipLaunchKernelGGL(k_adam, dim3((NPARAM + 255) / 256), dim3(256), 0, (hipStream_t)stream, t->w, t->m, t->v, t->grad,
                       lr, beta1, beta2, c1, c2, eps);
    return hip_status(hipGetLastError(), "Adam launch");
}

int mfc_trainer_infer(mfc_trainer *t, const uint16_t *features, int64_t n, float *prob, void *stream)
{
    if (!t || !features || !prob) return fail(MFC_E_ARG, "null argument");
    if (n < 1) return fail(MFC_E_ARG, "n must be >= 1");
    const int64_t tiles = (n + 15) / 16;
    const unsigned blocks = (unsigned)std::min<int64_t>((tiles + kWaves - 1) / kWaves, 4096);
    hipLaunchKernelGGL(k_mlp_infer, dim3(blocks), dim3(kThreads), 0, (hipStream_t)stream, t->w, features, n, prob);
    return hip_status(hipGetLastError(), "inference launch");
}

int mfc_set_indicator(mfc_grid *h, const float *params_host, double tau)
{
    if (!h || !params_host) return fail(MFC_E_ARG, "null argument");
    if (!std::isfinite(tau)) return fail(MFC_E_ARG, "tau must be finite");
    for (int i = 0; i < NPARAM; i++)
        if (!std::isfinite(params_host[i])) return fail(MFC_E_ARG, "non-finite network parameter");
    hipError_t e = hipSetDevice(h->device);
    if (e == hipSuccess && !h->mlp) e = hipMalloc((void **)&h->mlp, kRoutedWords * sizeof(float));
    if (e == hipSuccess) e = hipMemcpy(h->mlp, params_host, NPARAM * sizeof(float), hipMemcpyHostToDevice);
    if (e == hipSuccess) {
        // waited for before work of any stream reads it, on its own stream
        // only: other streams' work goes on
        hipLaunchKernelGGL(k_zero_logit, dim3(1), dim3(kThreads), 0, nullptr, h->mlp);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
    if (e != hipSuccess) return hip_status(e, "indicator upload");
    // P > tau  <=>  logit > log(tau / (1 - tau))
    h->logit_tau = tau <= 0.0 ? -INFINITY : (tau >= 1.0 ? INFINITY : (float)std::log(tau / (1.0 - tau)));
    return MFC_OK;
}

}  // extern "C"
