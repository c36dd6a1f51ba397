// Learned cost model of a work item: a 12 -> 64 -> 64 -> 1 ReLU perceptron in
// FP32 with hand-written forward, backward and Adam kernels.
//
// The paper observes that the computational weight of an element cannot be
// estimated a priori and that the number of Gauss points, used as the METIS
// weight, balances poorly (abstract; Section 4.1, Figures lb_resp/lb_iter).
// The batched assembly records the cycles every work item takes; this model
// learns log(cycles) from item features and orders the work queue.
//
// Layouts: parameters W1[64][12], b1[64], W2[64][64], b2[64], W3[64], b3;
// features row-major [n][12]; activations row-major [n][64].
// Gradients are reduced in a fixed order that depends on n alone (per wave its
// tiles of 16 samples in ascending order, then the waves, then the workgroups,
// the last in FP64), so training is deterministic.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <vector>

#include "fea_internal.h"

namespace fea {

constexpr int NI = 12, NH = 64;
constexpr int OW1 = 0, OB1 = OW1 + NH * NI, OW2 = OB1 + NH, OB2 = OW2 + NH * NH, OW3 = OB2 + NH,
              OB3 = OW3 + NH, NPAR = OB3 + 1;
static_assert(NPAR == FEA_COST_PARAMS, "parameter count");

// The layers are matrix products over the samples, done with FP32 matrix
// instructions (v_mfma_f32_16x16x4_f32: FP32 products and sums). A wave takes
// 16 samples through the forward pass, the backward pass and the parameter
// gradients by itself, its activations in LDS rows of its own and the whole
// gradient of the three layers in accumulators, so the only barriers are
// around the weights' load and the final sum over the workgroup's waves.
//
// Operand layout of the instruction: lane l holds A[l % 16][l / 16] and
// B[l / 16][l % 16] of a 16x4 and a 4x16 factor, and rows 4 (l / 16) + r,
// column l % 16 of the product. Row strides of 68 (activations, W2) and 20
// (inputs, W1) words put the 64 operands of one instruction in 64 different
// banks, except W2 read along its columns (about two per bank).
//
// Bound: the matrix instructions, 220 per 16 samples (7,040 cycles of one
// SIMD), 12 us for 60,000 samples. Measured on MI355X for 60,000 samples: a
// training step 37 us (this kernel 32, the sum with Adam 5), a prediction 11
// us; before, 573 and 105 us (one thread per sample in the forward and
// backward passes, activations through HBM, partial gradients of 64 samples, a
// 938-term sum per parameter on 20 workgroups). What is left beside the
// products is the start (weights to LDS) and the end (10 MB of partials) of
// workgroups that live for one or two tiles per wave.
constexpr int SW = 68, SX = 20;  // row strides in LDS
constexpr int WAVE_LDS = 2 * 16 * SW + 16 * SX;
constexpr int MLP_LDS = NH * SW + NH * SX + 3 * NH + 4 * WAVE_LDS;
constexpr int MAX_PART = 512;  // workgroups of a training step: two per CU
static_assert(MLP_LDS >= 3 * (NPAR + 1), "three waves' gradients are summed in the same LDS");

typedef float f32x4 __attribute__((ext_vector_type(4)));

// LDS written by other lanes of the wave may be read after this.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sample tiles of 16: wave w of workgroup b takes tiles 4 b + w, then every
// (4 gridDim)-th. TRAIN: part[b] receives the workgroup's gradient sums in
// parameter order and, after them, its sum of squared residuals; otherwise y
// receives the predictions.
template <bool TRAIN>
__global__ void __launch_bounds__(256, 2) k_mlp(const float *P, const float *mean, const float *scale, const float *X,
                                                const float *target, int64_t n, float *y, float *part)
{
    __shared__ __align__(16) float lds[MLP_LDS];
    float *sW2 = lds, *sW1 = sW2 + NH * SW, *sB1 = sW1 + NH * SX, *sB2 = sB1 + NH, *sW3 = sB2 + NH;
    const int tid = threadIdx.x, wave = tid >> 6, l = tid & 63, c = l & 15, kb = l >> 4;
    float *sH = sW3 + NH + wave * WAVE_LDS, *sD = sH + 16 * SW, *sZ = sD + 16 * SW;
    {
        // all loads before the first use: one memory latency
        f32x4 w2[4];
        float w1[3], v = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) w2[k] = reinterpret_cast<const f32x4 *>(P + OW2)[tid + 256 * k];
#pragma unroll
        for (int k = 0; k < 3; ++k) w1[k] = P[OW1 + tid + 256 * k];
        if (tid < 3 * NH) v = P[tid < NH ? OB1 + tid : tid < 2 * NH ? OB2 + tid - NH : OW3 + tid - 2 * NH];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = 4 * (tid + 256 * k);
            *reinterpret_cast<f32x4 *>(sW2 + (i / NH) * SW + i % NH) = w2[k];
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int i = tid + 256 * k;
            sW1[(i / NI) * SX + i % NI] = w1[k];
        }
        if (tid < 3 * NH) sB1[tid] = v;  // b1, b2, W3 back to back
    }
    const float b3 = P[OB3];
    const int zk = l & 15;  // this lane's input feature
    const float zm = zk < NI ? mean[zk] : 0.f, zs = zk < NI ? scale[zk] : 1.f;
    __syncthreads();
    float b1[4], b2[4], w3[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        b1[j] = sB1[16 * j + c];
        b2[j] = sB2[16 * j + c];
        w3[j] = sW3[16 * j + c];
    }
    f32x4 gW2[4][4], gW1[4];
    float gW3[4], gB2[4], gB1[4], gB3 = 0.f, loss = 0.f;
    if constexpr (TRAIN) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            gW1[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            gW3[i] = gB2[i] = gB1[i] = 0.f;
#pragma unroll
            for (int j = 0; j < 4; ++j) gW2[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    const int64_t tiles = (n + 15) / 16, step = (int64_t)gridDim.x * 4;
    // a tile's inputs and targets, at clamped positions (beyond n they are not
    // used), loaded one tile ahead
    float xn[4], tn[4] = {0.f, 0.f, 0.f, 0.f};
    auto fetch = [&](int64_t t0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t s = t0 * 16 + kb + 4 * i;
            xn[i] = X[(s < n ? s : n - 1) * NI + (zk < NI ? zk : 0)];
            if constexpr (TRAIN) {
                const int64_t q = t0 * 16 + 4 * kb + i;
                tn[i] = target[q < n ? q : n - 1];
            }
        }
    };
    fetch((int64_t)blockIdx.x * 4 + wave);
    for (int64_t t0 = (int64_t)blockIdx.x * 4 + wave; t0 < tiles; t0 += step) {
        const int64_t s0 = t0 * 16;
        // standardised inputs, columns 12 .. 15 zero
        float tv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int s = kb + 4 * i;
            sZ[s * SX + zk] = zk < NI && s0 + s < n ? (xn[i] - zm) / zs : 0.f;
            tv[i] = tn[i];
        }
        fetch(t0 + step);
        wave_lds_sync();
        f32x4 h1[4], h2[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            h1[j] = f32x4{b1[j], b1[j], b1[j], b1[j]};
            h2[j] = f32x4{b2[j], b2[j], b2[j], b2[j]};
        }
#pragma unroll
        for (int t = 0; t < NI / 4; ++t) {
            const float a = sZ[c * SX + 4 * t + kb];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                h1[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, sW1[(16 * j + c) * SX + 4 * t + kb], h1[j], 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                h1[j][r] = h1[j][r] > 0.f ? h1[j][r] : 0.f;
                sH[(4 * kb + r) * SW + 16 * j + c] = h1[j][r];
            }
        wave_lds_sync();
#pragma unroll 4
        for (int t = 0; t < NH / 4; ++t) {
            const float a = sH[c * SW + 4 * t + kb];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                h2[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, sW2[(16 * j + c) * SW + 4 * t + kb], h2[j], 0, 0, 0);
        }
        float out[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                h2[j][r] = h2[j][r] > 0.f ? h2[j][r] : 0.f;
                out[r] += w3[j] * h2[j][r];
            }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) out[r] += __shfl_xor(out[r], o);
            out[r] += b3;
        }
        if constexpr (!TRAIN) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (c == r && s0 + 4 * kb + r < n) y[s0 + 4 * kb + r] = out[r];
        } else {
            // dy = 2 (y - t) / n, dA2 = dy W3 (.) [h2 > 0]
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool ok = s0 + 4 * kb + r < n;
                const float res = ok ? out[r] - tv[r] : 0.f, dy = ok ? 2.f * res / (float)n : 0.f;
                loss += res * res;
                gB3 += dy;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float d = h2[j][r] > 0.f ? dy * w3[j] : 0.f;
                    gW3[j] += dy * h2[j][r];
                    gB2[j] += d;
                    sD[(4 * kb + r) * SW + 16 * j + c] = d;
                }
            }
            wave_lds_sync();
            // dA1 = (dA2 W2) (.) [h1 > 0]
            f32x4 d1[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) d1[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
            for (int t = 0; t < NH / 4; ++t) {
                const float a = sD[c * SW + 4 * t + kb];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    d1[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, sW2[(4 * t + kb) * SW + 16 * j + c], d1[j], 0, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    d1[j][r] = h1[j][r] > 0.f ? d1[j][r] : 0.f;
                    gB1[j] += d1[j][r];
                }
            // gradient of W2: sum over the samples of dA2 (x) h1
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                float a[4], b[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    a[j] = sD[(t + 4 * kb) * SW + 16 * j + c];
                    b[j] = sH[(t + 4 * kb) * SW + 16 * j + c];
                }
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        gW2[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], gW2[i][j], 0, 0, 0);
            }
            wave_lds_sync();
            // and of W1: dA1 (x) z, dA1 in the place of h1
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) sH[(4 * kb + r) * SW + 16 * j + c] = d1[j][r];
            wave_lds_sync();
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float b = sZ[(t + 4 * kb) * SX + c];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    gW1[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(sH[(t + 4 * kb) * SW + 16 * i + c], b, gW1[i], 0, 0, 0);
            }
        }
        wave_lds_sync();  // the tile's rows are no longer read
    }
    if constexpr (TRAIN) {
        // the vectors' sums over the lanes' four row groups; b3 and the loss
        // are the same in the 16 lanes of a row group
#pragma unroll
        for (int o = 16; o < 64; o <<= 1) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                gW3[j] += __shfl_xor(gW3[j], o);
                gB2[j] += __shfl_xor(gB2[j], o);
                gB1[j] += __shfl_xor(gB1[j], o);
            }
            gB3 += __shfl_xor(gB3, o);
            loss += __shfl_xor(loss, o);
        }
        // waves 1 .. 3 to regions of their own, wave 0 added to wave 1's, then
        // the sum of the three
        float *mine = lds + (wave ? wave - 1 : 0) * (NPAR + 1);
        auto put = [&](bool add) {
            auto at = [&](int p, float v) { mine[p] = add ? v + mine[p] : v; };
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int u = 16 * i + 4 * kb + r;
                    if (c < NI) at(OW1 + u * NI + c, gW1[i][r]);
#pragma unroll
                    for (int j = 0; j < 4; ++j) at(OW2 + u * NH + 16 * j + c, gW2[i][j][r]);
                }
            if (kb == 0) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    at(OB1 + 16 * j + c, gB1[j]);
                    at(OB2 + 16 * j + c, gB2[j]);
                    at(OW3 + 16 * j + c, gW3[j]);
                }
            }
            if (l == 0) {
                at(OB3, gB3);
                at(NPAR, loss);
            }
        };
        __syncthreads();
        if (wave) put(false);
        __syncthreads();
        if (!wave) put(true);
        __syncthreads();
        for (int p = tid; p <= NPAR; p += 256)
            part[(int64_t)blockIdx.x * (NPAR + 1) + p] = lds[p] + lds[NPAR + 1 + p] + lds[2 * (NPAR + 1) + p];
    }
}

// Sum of the workgroups' partials in FP64, 64 parameters per workgroup: wave w
// of 16 takes rows w, w + 16, ... in order, then the 16 sums are added in
// order. grad and loss (sum r^2 / n) may be NULL; ADAM: the parameters' step
// with this gradient.
struct AdamArgs {
    float *P, *m, *v;
    float lr, b1, b2, eps, c1, c2;
};

template <bool ADAM>
__global__ void __launch_bounds__(1024) k_mlp_reduce(const float *part, int rows, int64_t n, float *grad, float *loss,
                                                     AdamArgs A)
{
    __shared__ double sum[16][64];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, p = blockIdx.x * 64 + l;
    double acc = 0.0;
    if (p <= NPAR) {
#pragma unroll 8
        for (int r = w; r < rows; r += 16) acc += (double)part[(int64_t)r * (NPAR + 1) + p];
    }
    sum[w][l] = acc;
    __syncthreads();
    if (w || p > NPAR) return;
#pragma unroll
    for (int k = 1; k < 16; ++k) acc += sum[k][l];
    if (p == NPAR) {
        if (loss) *loss = (float)acc / (float)n;
        return;
    }
    const float g = (float)acc;
    if (grad) grad[p] = g;
    if constexpr (ADAM) {
        const float mp = A.b1 * A.m[p] + (1.f - A.b1) * g;
        const float vp = A.b2 * A.v[p] + (1.f - A.b2) * g * g;
        A.m[p] = mp;
        A.v[p] = vp;
        A.P[p] -= A.lr * (mp / A.c1) / (sqrtf(vp / A.c2) + A.eps);
    }
}

// Per-feature mean and population standard deviation, in FP64 and a fixed
// order: thread t of workgroup b sums elements 252 b + t + k * 252 * gridDim of
// the row-major features (252 = 21 rows, so an element's feature is t % 12),
// the workgroup its 21 threads of a feature, the last kernel the workgroups.
// 11 us for 60,000 samples; with one workgroup per feature (12 of 256 CUs) 68.
constexpr int NORM_T = 21 * NI, NORM_WG = 128;

__global__ void __launch_bounds__(256) k_norm_part(const float *X, int64_t n, double *part)
{
    __shared__ double s1[NORM_T], s2[NORM_T];
    const int t = threadIdx.x;
    if (t < NORM_T) {
        double a = 0.0, b = 0.0;
        for (int64_t i = (int64_t)blockIdx.x * NORM_T + t; i < n * NI; i += (int64_t)gridDim.x * NORM_T) {
            const double x = X[i];
            a += x;
            b += x * x;
        }
        s1[t] = a;
        s2[t] = b;
    }
    __syncthreads();
    if (t < 2 * NI) {
        const double *s = t < NI ? s1 : s2;
        double a = 0.0;
        for (int r = 0; r < 21; ++r) a += s[r * NI + t % NI];
        part[blockIdx.x * 2 * NI + t] = a;
    }
}

constexpr int NORM_SEG = 32;

__global__ void __launch_bounds__(2 * NI * NORM_SEG) k_norm_final(const double *part, int rows, int64_t n, float *mean,
                                                                  float *scale)
{
    __shared__ double s[NORM_SEG][2 * NI];
    const int c = threadIdx.x % (2 * NI), seg = threadIdx.x / (2 * NI);
    double a = 0.0;
    for (int r = seg; r < rows; r += NORM_SEG) a += part[r * 2 * NI + c];
    s[seg][c] = a;
    __syncthreads();
    const int k = threadIdx.x;
    if (k >= NI) return;
    double s1 = 0.0, s2 = 0.0;
    for (int r = 0; r < NORM_SEG; ++r) {
        s1 += s[r][k];
        s2 += s[r][NI + k];
    }
    const double mu = s1 / (double)n;
    const double var = std::max(0.0, s2 / (double)n - mu * mu);
    const double sd = sqrt(var);
    mean[k] = (float)mu;
    scale[k] = sd > 1e-12 ? (float)sd : 1.f;
}

__global__ void k_log_cycles(const uint64_t *c, int64_t n, float *t)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) t[i] = logf((float)(c[i] > 0 ? c[i] : 1));
}

}  // namespace fea

using namespace fea;

struct fea_cost {
    int device = 0;
    float *P = nullptr, *m = nullptr, *v = nullptr, *mean = nullptr, *scale = nullptr;
    double *norm = nullptr;  // partial sums of fit_norm
    int64_t step = 0;
    // partial gradients, one row of NPAR + 1 per workgroup
    float *ws = nullptr;
    int64_t ws_rows = 0;
};

namespace {

uint64_t splitmix(uint64_t &x)
{
    uint64_t z = (x += 0x9e3779b97f4a7c15ull);
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

// standard normal by Box-Muller from a SplitMix64 stream
double normal(uint64_t &x)
{
    const double u1 = ((splitmix(x) >> 11) + 1.0) * 0x1.0p-53;
    const double u2 = (splitmix(x) >> 11) * 0x1.0p-53;
    return sqrt(-2.0 * log(u1)) * cos(2.0 * M_PI * u2);
}

void destroy_cost(fea_cost *c)
{
    if (!c) return;
    dfree(c->P);  // with it m, v, mean, scale and norm
    dfree(c->ws);
    delete c;
}

// Workgroups of a training step over n samples (four waves of 16 samples).
int64_t part_rows(int64_t n) { return std::min<int64_t>(MAX_PART, (n + 63) / 64); }

int ensure_ws(fea_cost *c, int64_t n)
{
    const int64_t rows = part_rows(n);
    if (c->ws && c->ws_rows >= rows) return FEA_OK;
    dfree(c->ws);
    c->ws = nullptr;
    c->ws_rows = 0;
    int rc = dalloc((void **)&c->ws, sizeof(float) * (size_t)rows * (NPAR + 1));
    if (rc) return rc;
    c->ws_rows = rows;
    return FEA_OK;
}

// One pass over the samples and the sum of its partials; with adam, the step.
int grad_impl(const fea_cost *c, const float *X, const float *t, int64_t n, float *grad, float *loss,
              const AdamArgs *adam, hipStream_t s)
{
    const int rows = (int)part_rows(n);
    k_mlp<true><<<rows, 256, 0, s>>>(c->P, c->mean, c->scale, X, t, n, nullptr, c->ws);
    const unsigned nb = grid_for(NPAR + 1, 64);
    if (adam)
        k_mlp_reduce<true><<<nb, 1024, 0, s>>>(c->ws, rows, n, grad, loss, *adam);
    else
        k_mlp_reduce<false><<<nb, 1024, 0, s>>>(c->ws, rows, n, grad, loss, AdamArgs());
    FEA_HIP(hipGetLastError());
    return FEA_OK;
}

int check(const fea_cost *c)
{
    if (!c) return set_error(FEA_EINVAL, "cost model is NULL");
    int dev = 0;
    FEA_HIP(hipGetDevice(&dev));
    if (dev != c->device) return set_error(FEA_EINVAL, "cost model lives on device %d", c->device);
    return FEA_OK;
}

const char kMagic[8] = {'F', 'E', 'A', 'C', 'O', 'S', 'T', '1'};
const char kArch[8] = {'g', 'f', 'x', '9', '5', '0', 0, 0};
const uint32_t kVersion = 1;

}  // namespace

extern "C" int fea_cost_create(uint64_t seed, fea_cost **out)
{
    clear_error();
    if (!out) return set_error(FEA_EINVAL, "out is NULL");
    *out = nullptr;
    fea_cost *c = new (std::nothrow) fea_cost();
    if (!c) return set_error(FEA_ENOMEM, "host allocation failed");
    (void)hipGetDevice(&c->device);
    // one block: parameters, Adam moments, standardisation, partial sums
    constexpr size_t PP = (NPAR + 63) / 64 * 64, HEAD = 3 * PP + 64;
    int rc = dalloc((void **)&c->P, sizeof(float) * HEAD + sizeof(double) * NORM_WG * 2 * NI);
    if (rc) {
        destroy_cost(c);
        return rc;
    }
    c->m = c->P + PP;
    c->v = c->m + PP;
    c->mean = c->v + PP;
    c->scale = c->mean + 32;
    c->norm = reinterpret_cast<double *>(c->P + HEAD);
    std::vector<float> P(HEAD, 0.f);
    uint64_t st = seed;
    for (int i = 0; i < NH * NI; ++i) P[OW1 + i] = (float)(normal(st) * sqrt(2.0 / NI));
    for (int i = 0; i < NH * NH; ++i) P[OW2 + i] = (float)(normal(st) * sqrt(2.0 / NH));
    for (int i = 0; i < NH; ++i) P[OW3 + i] = (float)(normal(st) * sqrt(2.0 / NH));
    std::fill(P.begin() + 3 * PP + 32, P.begin() + 3 * PP + 32 + NI, 1.f);
    hipError_t e = hipMemcpy(c->P, P.data(), sizeof(float) * HEAD, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        destroy_cost(c);
        return set_error(FEA_EHIP, "upload failed: %s", hipGetErrorString(e));
    }
    *out = c;
    return FEA_OK;
}

extern "C" void fea_cost_destroy(fea_cost *c) { destroy_cost(c); }

extern "C" int fea_cost_get_params(const fea_cost *c, float *params)
{
    clear_error();
    if (!c || !params) return set_error(FEA_EINVAL, "cost model and params are required");
    FEA_HIP(hipMemcpy(params, c->P, sizeof(float) * NPAR, hipMemcpyDeviceToHost));
    return FEA_OK;
}

extern "C" int fea_cost_set_params(fea_cost *c, const float *params)
{
    clear_error();
    if (!c || !params) return set_error(FEA_EINVAL, "cost model and params are required");
    FEA_HIP(hipMemcpy(c->P, params, sizeof(float) * NPAR, hipMemcpyHostToDevice));
    return FEA_OK;
}

extern "C" int fea_cost_set_norm(fea_cost *c, const float *mean, const float *scale)
{
    clear_error();
    if (!c || !mean || !scale) return set_error(FEA_EINVAL, "cost model, mean and scale are required");
    for (int k = 0; k < NI; ++k)
        if (!(scale[k] > 0.f)) return set_error(FEA_EINVAL, "scale[%d] must be positive", k);
    FEA_HIP(hipMemcpy(c->mean, mean, sizeof(float) * NI, hipMemcpyHostToDevice));
    FEA_HIP(hipMemcpy(c->scale, scale, sizeof(float) * NI, hipMemcpyHostToDevice));
    return FEA_OK;
}

extern "C" int fea_cost_fit_norm(fea_cost *c, const float *feats, int64_t n, hipStream_t s)
{
    clear_error();
    int rc = check(c);
    if (rc) return rc;
    if (n <= 0 || !feats) return set_error(FEA_EINVAL, "need features");
    const int rows = (int)std::min<int64_t>(NORM_WG, (n + 20) / 21);
    k_norm_part<<<rows, 256, 0, s>>>(feats, n, c->norm);
    k_norm_final<<<1, 2 * NI * NORM_SEG, 0, s>>>(c->norm, rows, n, c->mean, c->scale);
    FEA_HIP(hipGetLastError());
    return FEA_OK;
}

extern "C" int fea_cost_predict(const fea_cost *c, const float *feats, int64_t n, float *pred, hipStream_t s)
{
    clear_error();
    int rc = check(c);
    if (rc) return rc;
    if (n < 0 || (n > 0 && (!feats || !pred))) return set_error(FEA_EINVAL, "bad arguments");
    if (n)
        k_mlp<false><<<(unsigned)std::min<int64_t>(2 * MAX_PART, (n + 63) / 64), 256, 0, s>>>(
            c->P, c->mean, c->scale, feats, nullptr, n, pred, nullptr);
    FEA_HIP(hipGetLastError());
    return FEA_OK;
}

extern "C" int fea_cost_grad(const fea_cost *c, const float *feats, const float *target, int64_t n,
                             float *grad, float *loss, hipStream_t s)
{
    clear_error();
    int rc = check(c);
    if (rc) return rc;
    if (n <= 0 || !feats || !target) return set_error(FEA_EINVAL, "bad arguments");
    if ((rc = ensure_ws(const_cast<fea_cost *>(c), n))) return rc;
    return grad_impl(c, feats, target, n, grad, loss, nullptr, s);
}

extern "C" int fea_cost_train(fea_cost *c, const float *feats, const float *target, int64_t n, int steps,
                              float lr, float *loss_hist, hipStream_t s)
{
    clear_error();
    int rc = check(c);
    if (rc) return rc;
    if (n <= 0 || steps < 0 || !feats || !target || !(lr > 0.f)) return set_error(FEA_EINVAL, "bad arguments");
    if ((rc = ensure_ws(c, n))) return rc;
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    for (int k = 0; k < steps; ++k) {
        const float c1 = 1.f - powf(b1, (float)(c->step + 1)), c2 = 1.f - powf(b2, (float)(c->step + 1));
        const AdamArgs adam = {c->P, c->m, c->v, lr, b1, b2, eps, c1, c2};
        if ((rc = grad_impl(c, feats, target, n, nullptr, loss_hist ? loss_hist + k : nullptr, &adam, s))) return rc;
        c->step += 1;
    }
    return FEA_OK;
}

extern "C" int fea_cost_log_cycles(const uint64_t *cycles, int64_t n, float *target, hipStream_t s)
{
    clear_error();
    if (n < 0 || (n > 0 && (!cycles || !target))) return set_error(FEA_EINVAL, "bad arguments");
    if (n) k_log_cycles<<<grid_for(n, 256), 256, 0, s>>>(cycles, n, target);
    FEA_HIP(hipGetLastError());
    return FEA_OK;
}

extern "C" int fea_cost_save(const fea_cost *c, const char *path)
{
    clear_error();
    if (!c || !path) return set_error(FEA_EINVAL, "cost model and path are required");
    std::vector<float> P(NPAR), m(NPAR), v(NPAR), mean(NI), scale(NI);
    FEA_HIP(hipDeviceSynchronize());
    FEA_HIP(hipMemcpy(P.data(), c->P, sizeof(float) * NPAR, hipMemcpyDeviceToHost));
    FEA_HIP(hipMemcpy(m.data(), c->m, sizeof(float) * NPAR, hipMemcpyDeviceToHost));
    FEA_HIP(hipMemcpy(v.data(), c->v, sizeof(float) * NPAR, hipMemcpyDeviceToHost));
    FEA_HIP(hipMemcpy(mean.data(), c->mean, sizeof(float) * NI, hipMemcpyDeviceToHost));
    FEA_HIP(hipMemcpy(scale.data(), c->scale, sizeof(float) * NI, hipMemcpyDeviceToHost));
    FILE *f = fopen(path, "wb");
    if (!f) return set_error(FEA_EINVAL, "cannot write %s", path);
    bool ok = fwrite(kMagic, 1, 8, f) == 8 && fwrite(&kVersion, 4, 1, f) == 1 && fwrite(kArch, 1, 8, f) == 8 &&
              fwrite(mean.data(), 4, NI, f) == NI && fwrite(scale.data(), 4, NI, f) == NI &&
              fwrite(P.data(), 4, NPAR, f) == NPAR && fwrite(m.data(), 4, NPAR, f) == NPAR &&
              fwrite(v.data(), 4, NPAR, f) == NPAR && fwrite(&c->step, 8, 1, f) == 1;
    fclose(f);
    if (!ok) return set_error(FEA_EINVAL, "short write to %s", path);
    return FEA_OK;
}

extern "C" int fea_cost_load(fea_cost *c, const char *path)
{
    clear_error();
    if (!c || !path) return set_error(FEA_EINVAL, "cost model and path are required");
    FILE *f = fopen(path, "rb");
    if (!f) return set_error(FEA_EINVAL, "cannot read %s", path);
    char magic[8], arch[8];
    uint32_t ver = 0;
    std::vector<float> P(NPAR), m(NPAR), v(NPAR), mean(NI), scale(NI);
    int64_t step = 0;
    bool ok = fread(magic, 1, 8, f) == 8 && fread(&ver, 4, 1, f) == 1 && fread(arch, 1, 8, f) == 8 &&
              fread(mean.data(), 4, NI, f) == NI && fread(scale.data(), 4, NI, f) == NI &&
              fread(P.data(), 4, NPAR, f) == NPAR && fread(m.data(), 4, NPAR, f) == NPAR &&
              fread(v.data(), 4, NPAR, f) == NPAR && fread(&step, 8, 1, f) == 1;
    fclose(f);
    if (!ok || memcmp(magic, kMagic, 8) != 0 || ver != kVersion || memcmp(arch, kArch, 8) != 0)
        return set_error(FEA_EINVAL, "%s is not a cost-model checkpoint of this version", path);
    FEA_HIP(hipMemcpy(c->P, P.data(), sizeof(float) * NPAR, hipMemcpyHostToDevice));
    FEA_HIP(hipMemcpy(c->m, m.data(), sizeof(float) * NPAR, hipMemcpyHostToDevice));
    FEA_HIP(hipMemcpy(c->v, v.data(), sizeof(float) * NPAR, hipMemcpyHostToDevice));
    FEA_HIP(hipMemcpy(c->mean, mean.data(), sizeof(float) * NI, hipMemcpyHostToDevice));
    FEA_HIP(hipMemcpy(c->scale, scale.data(), sizeof(float) * NI, hipMemcpyHostToDevice));
    c->step = step;
    return FEA_OK;
}
