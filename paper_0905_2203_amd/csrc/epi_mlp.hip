// Cost model of the scheduler: a perceptron with two hidden ReLU layers of
// 64 units, FP32, trained on the mean squared error with Adam, entirely on
// the device.
//
//   h1 = relu(x W1 + b1), h2 = relu(h1 W2 + b2), y = h2 w3 + b3
//   L  = mean_i (y_i - t_i)^2
//
// Parameters: one flat FP32 vector W1[F][64], b1[64], W2[64][64], b2[64],
// w3[64], b3[1].
//
// k_mlp_rows:   one wave per tile of 4 or 8 samples, lane j = hidden unit j: the
//   forward pass and, when training, the back-propagated terms and the tile's
//   gradient, added up over the wave's tiles in a part of its own.
// k_mlp_sum:    sums the parts of each parameter's gradient in a fixed order
//   (deterministic) and, in a training step, applies Adam step k.
// k_mlp_adam:   one thread per parameter; Adam step k with a given gradient.
// k_standardize, k_affine_base: the cost model's input and output scaling
//   around the network, (x - mu) * isd per feature and y * sd + mu, plus the
//   raw base feature (the network predicts the correction to it).
#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "epi_internal.h"

namespace epi {

namespace {

constexpr int kH = kMlpHidden;

__host__ __device__ inline int64_t n_params_of(int F) { return (int64_t)F * kH + kH + kH * kH + kH + kH + 1; }

// What bounds a training step is latency: 512 samples are 9 million multiply-adds,
// nothing for the chip, in a chain of forward, backward, gradient and update.  One
// thread a sample with all weights broadcast from LDS (79 us), then one thread a
// parameter summing 512 samples in a row (134 us), then the loss fetched by the
// host took 262 us a step; a wave a tile spreads the batch over 128 waves and
// leaves sums of at most kParts / 4 a thread: 14 + 4 us a step (an epoch of 16
// steps of 512 and 50k predictions, host copies included: 4.2 -> 0.69 ms).
//
// A training step's sums are FP64 (the parameters, moments and inputs FP32): Adam
// divides a gradient by its own size, so where a parameter's gradient all but
// cancels, the sums' rounding moves it by up to the learning rate.  With other
// FP32 sums than a serial run's, the predictions of 1 epoch in some 10 were
// further from exact ones than that run's; so they are as near or nearer in all
// of 24 (0.63 -> 0.69 ms).
constexpr int kMlpWaves = 4;     // waves per workgroup, sharing the staged W2
constexpr int kParts = 256;      // most gradient parts (waves of a training launch)
constexpr int kRow = kH + 1;     // W2's row in LDS: rows and columns free of bank conflicts

// y[s] for every sample; TRAIN also the gradient parts part[wave][n_params] of
// the loss over B samples, and the squared errors.  S samples a tile.
template <bool TRAIN, int S>
__global__ __launch_bounds__(64 * kMlpWaves) void k_mlp_rows(const float *__restrict__ p, int F,
                                                             const float *__restrict__ X, const float *__restrict__ t,
                                                             int64_t B, float *__restrict__ y, double *__restrict__ part,
                                                             float *__restrict__ sqerr) {
    using A = std::conditional_t<TRAIN, double, float>;
    __shared__ float W2[kH * kRow];
    __shared__ __align__(16) float W1s[kH * kH];  // W1, for up to 64 inputs
    __shared__ __align__(16) float xb[kMlpWaves][kH][S];  // 64 inputs of the tile's samples
    __shared__ __align__(16) A hb[kMlpWaves][kH][S];      // h1
    __shared__ __align__(16) A db[TRAIN ? kMlpWaves : 1][kH][S];  // dz2
    const int j = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const float *W1 = p, *b1 = p + (int64_t)F * kH, *pW2 = b1 + kH, *b2 = pW2 + kH * kH, *w3 = b2 + kH, *b3 = w3 + kH;
    float(*x)[S] = xb[wv];
    A(*h)[S] = hb[wv], (*d)[S] = db[TRAIN ? wv : 0];
    const float vb1 = b1[j], vb2 = b2[j], vw3 = w3[j], vb3 = b3[0];
    const bool staged = F <= kH;
    {
        // all loads in flight together (the rows start on 16 bytes)
        constexpr int kN = kH * kH / (4 * 64 * kMlpWaves);
        float4 a[kN], b[kN];
        const int nw1 = staged ? F * kH / 4 : 0;
#pragma unroll
        for (int r = 0; r < kN; ++r) {
            const int i = r * 64 * kMlpWaves + (int)threadIdx.x;
            a[r] = reinterpret_cast<const float4 *>(pW2)[i];
            b[r] = i < nw1 ? reinterpret_cast<const float4 *>(W1)[i] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int r = 0; r < kN; ++r) {
            const int i = r * 64 * kMlpWaves + (int)threadIdx.x;
            float *o = W2 + (i / (kH / 4)) * kRow + (i % (kH / 4)) * 4;
            o[0] = a[r].x;
            o[1] = a[r].y;
            o[2] = a[r].z;
            o[3] = a[r].w;
            reinterpret_cast<float4 *>(W1s)[i] = b[r];
        }
    }
    __syncthreads();  // (the only barrier: from here on the waves work alone)
    const int64_t wave = (int64_t)blockIdx.x * kMlpWaves + wv, waves = (int64_t)gridDim.x * kMlpWaves;
    double *g = TRAIN ? part + wave * n_params_of(F) : nullptr;
    bool first = true;
    for (int64_t s0 = wave * S; s0 < B; s0 += waves * S) {
        const int ns = B - s0 < S ? (int)(B - s0) : S;
        // inputs f0 .. f0+63 of the tile (zero for the samples past the batch)
        auto stage = [&](int f0) {
            __builtin_amdgcn_wave_barrier();
            float v[S];
            const int f = f0 + j < F ? f0 + j : F - 1;
#pragma unroll
            for (int q = 0; q < S; ++q) v[q] = X[(s0 + (q < ns ? q : 0)) * F + f];
#pragma unroll
            for (int q = 0; q < S; ++q) x[j][q] = q < ns && f0 + j < F ? v[q] : 0.f;
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
        };
        A h1[S], z2[S], out[S];
        float tq[S];
#pragma unroll
        for (int q = 0; q < S; ++q) {
            h1[q] = vb1;
            tq[q] = TRAIN && q < ns ? t[s0 + q] : 0.f;
        }
        for (int f0 = 0; f0 < F; f0 += kH) {
            stage(f0);
            const int nf = F - f0 < kH ? F - f0 : kH;
            auto column = [&](const float *w1) {
#pragma unroll 8
                for (int f = 0; f < nf; ++f) {
                    const A wt = w1[f * kH + j];
#pragma unroll
                    for (int q = 0; q < S; ++q) h1[q] = fma((A)x[f][q], wt, h1[q]);
                }
            };
            if (staged) column(W1s);
            else column(W1 + (int64_t)f0 * kH);
        }
#pragma unroll
        for (int q = 0; q < S; ++q) {
            h1[q] = h1[q] > 0 ? h1[q] : 0;  // z1 > 0 <=> h1 > 0
            h[j][q] = h1[q];
            z2[q] = vb2;
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll 8
        for (int a = 0; a < kH; ++a) {
            const A wt = W2[a * kRow + j];
#pragma unroll
            for (int q = 0; q < S; ++q) z2[q] = fma(h[a][q], wt, z2[q]);
        }
#pragma unroll
        for (int q = 0; q < S; ++q) {
            A v = z2[q] > 0 ? z2[q] * (A)vw3 : 0;
            for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
            out[q] = v + vb3;
            if (j == q && q < ns) y[s0 + q] = (float)out[q];
        }
        if constexpr (TRAIN) {
            // dz2 = dy * w3 * [z2 > 0];  dz1 = (dz2 W2^T) * [z1 > 0]
            A gb1 = 0, gb2 = 0, gw3 = 0, gb3 = 0, dz1[S], dz2[S];
#pragma unroll
            for (int q = 0; q < S; ++q) {
                const A r = q < ns ? out[q] - (A)tq[q] : 0;
                if (j == q && q < ns) sqerr[s0 + q] = (float)(r * r);
                const A dy = 2 * r / (A)B;
                dz2[q] = z2[q] > 0 ? dy * (A)vw3 : 0;
                gw3 = fma(z2[q] > 0 ? z2[q] : 0, dy, gw3);
                gb2 += dz2[q];
                gb3 += dy;
                d[j][q] = dz2[q];
                dz1[q] = 0;
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll 8
            for (int k = 0; k < kH; ++k) {  // lane j = unit j of the first layer
                const A wt = W2[j * kRow + k];
#pragma unroll
                for (int q = 0; q < S; ++q) dz1[q] = fma(d[k][q], wt, dz1[q]);
            }
#pragma unroll
            for (int q = 0; q < S; ++q) {
                dz1[q] = h1[q] > 0 ? dz1[q] : 0;
                gb1 += dz1[q];
            }
            // the tile's gradient onto the wave's part (each lane its own parameters)
            auto put = [&](int64_t o, A v) { g[o] = first ? v : g[o] + v; };
            for (int f0 = 0; f0 < F; f0 += kH) {
                if (F > kH) stage(f0);  // (else the inputs are still there)
                const int nf = F - f0 < kH ? F - f0 : kH;
#pragma unroll 4
                for (int f = 0; f < nf; ++f) {  // W1[f][j]: x_f dz1_j
                    A v = 0;
#pragma unroll
                    for (int q = 0; q < S; ++q) v = fma((A)x[f][q], dz1[q], v);
                    put((int64_t)(f0 + f) * kH + j, v);
                }
            }
            const int64_t o1 = (int64_t)F * kH;
            put(o1 + j, gb1);
#pragma unroll 4
            for (int a = 0; a < kH; ++a) {  // W2[a][j]: h1_a dz2_j
                A v = 0;
#pragma unroll
                for (int q = 0; q < S; ++q) v = fma(h[a][q], dz2[q], v);
                put(o1 + kH + a * kH + j, v);
            }
            const int64_t o2 = o1 + kH + kH * kH;
            put(o2 + j, gb2);
            put(o2 + kH + j, gw3);
            if (j == 0) put(o2 + 2 * kH, gb3);
            first = false;
        }
        __builtin_amdgcn_wave_barrier();
    }
}

__device__ __forceinline__ void adam(float *__restrict__ p, float *__restrict__ m, float *__restrict__ v, int64_t q,
                                     float gq, float lr, float b1, float b2, float eps, float c1, float c2) {
    const float mq = b1 * m[q] + (1.f - b1) * gq;
    const float vq = b2 * v[q] + (1.f - b2) * gq * gq;
    m[q] = mq;
    v[q] = vq;
    p[q] -= lr * (mq / c1) / (sqrtf(vq / c2) + eps);
}

// g = the sum of the parts, four threads a parameter, each over every fourth
// part; ADAM: and the step with it.
template <bool ADAM>
__global__ __launch_bounds__(256) void k_mlp_sum(const double *__restrict__ part, int parts, int64_t n,
                                                 float *__restrict__ g, float *__restrict__ p, float *__restrict__ m,
                                                 float *__restrict__ v, float lr, float b1, float b2, float eps,
                                                 float c1, float c2) {
    __shared__ double sum[4][64];
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t q = (int64_t)blockIdx.x * 64 + l;
    double acc = 0;
    if (q < n) {
#pragma unroll 16
        for (int i = w; i < parts; i += 4) acc += part[i * n + q];
    }
    sum[w][l] = acc;
    __syncthreads();
    if (w != 0 || q >= n) return;
    acc = (sum[0][l] + sum[1][l]) + (sum[2][l] + sum[3][l]);
    g[q] = (float)acc;
    if constexpr (ADAM) adam(p, m, v, q, (float)acc, lr, b1, b2, eps, c1, c2);
}

__global__ void k_mlp_adam(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                           float *__restrict__ v, int64_t n, float lr, float b1, float b2, float eps, float c1,
                           float c2) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    adam(p, m, v, q, g[q], lr, b1, b2, eps, c1, c2);
}

__global__ void k_standardize(float *__restrict__ X, int64_t n, int F, const float *__restrict__ norm) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    const int f = (int)(q % F);
    X[q] = (X[q] - norm[f]) * norm[F + f];
}

// y = y * sd + mu + x_base, where x_base is the raw value of input feature
// `base` of the sample (recovered from the standardised Xs: x = x' / isd + mu;
// a constant feature, isd = 0, is its mean); base < 0: no base term.
__global__ void k_affine_base(float *__restrict__ y, int64_t n, float sd, float mu, const float *__restrict__ Xs,
                              int F, const float *__restrict__ norm, int base) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    float b = 0.f;
    if (base >= 0) {
        const float isd = norm[F + base], m = norm[base];
        b = isd > 0.f ? Xs[q * F + base] / isd + m : m;
    }
    y[q] = fmaf(y[q], sd, mu) + b;
}

}  // namespace

int64_t mlp_n_params(int F) { return n_params_of(F); }

hipError_t mlp_set_scaling(Mlp &net, const float *x_mu, const float *x_isd, float y_mu, float y_sd) {
    net.x_mu.assign(x_mu, x_mu + net.F);
    net.x_isd.assign(x_isd, x_isd + net.F);
    net.y_mu = y_mu;
    net.y_sd = y_sd;
    std::vector<float> h(net.x_mu);
    h.insert(h.end(), net.x_isd.begin(), net.x_isd.end());
    hipError_t e;
    if (!net.norm.p && (e = net.norm.alloc(sizeof(float) * 2 * net.F)) != hipSuccess) return e;
    return hipMemcpy(net.norm.p, h.data(), sizeof(float) * h.size(), hipMemcpyHostToDevice);
}

hipError_t costmodel_predict_device(Mlp &net, float *dX, int64_t B, float *dy, hipStream_t st) {
    if (B == 0) return hipSuccess;
    const int64_t n = B * net.F;
    k_standardize<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(dX, n, net.F, net.norm.as<float>());
    hipError_t e;
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = mlp_forward_device(net, dX, B, dy, st)) != hipSuccess) return e;
    k_affine_base<<<(unsigned)((B + 255) / 256), 256, 0, st>>>(dy, B, net.y_sd, net.y_mu, dX, net.F,
                                                                net.norm.as<float>(),
                                                                net.F > kBaseFeature ? kBaseFeature : -1);
    return hipGetLastError();
}

// The inputs a model may have on the device: its parameters in 64 KiB of LDS.
// (The kernels need less; the bound keeps what a model accepts.)
static bool mlp_fits(const Mlp &net) { return sizeof(float) * (size_t)n_params_of(net.F) <= 64 * 1024; }

hipError_t mlp_forward_device(Mlp &net, const float *dX, int64_t B, float *dy, hipStream_t st) {
    if (B == 0) return hipSuccess;
    if (!mlp_fits(net)) return hipErrorInvalidValue;
    constexpr int S = 8;
    const int64_t tiles = (B + S - 1) / S, blocks = (tiles + kMlpWaves - 1) / kMlpWaves;
    // (staging W2 is amortised over a wave's tiles: no more workgroups than the chip holds)
    k_mlp_rows<false, S><<<(unsigned)std::min<int64_t>(blocks, 1024), 64 * kMlpWaves, 0, st>>>(
        net.p.as<float>(), net.F, dX, nullptr, B, dy, nullptr, nullptr);
    return hipGetLastError();
}

// Gradient over B device samples into dg, the squared errors into sq (device);
// step: then the Adam step with it.
static hipError_t grad_launch(Mlp &net, const float *dX, const float *dt, int64_t B, float *dg, float *sq, bool step,
                              hipStream_t st) {
    hipError_t e;
    if (!mlp_fits(net)) return hipErrorInvalidValue;
    constexpr int S = 4;
    const int64_t np = n_params_of(net.F);
    const size_t need = sizeof(double) * (size_t)kParts * np + sizeof(float) * (size_t)B;
    if (net.act.bytes < need) {
        if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
        if ((e = net.act.alloc(need)) != hipSuccess) return e;
    }
    double *part = net.act.as<double>();
    float *ys = reinterpret_cast<float *>(part + (size_t)kParts * np);
    const int64_t tiles = (B + S - 1) / S;
    const unsigned blocks = (unsigned)std::min<int64_t>((tiles + kMlpWaves - 1) / kMlpWaves, kParts / kMlpWaves);
    // (a wave without a tile writes no part)
    const int parts = (int)std::min<int64_t>(tiles, (int64_t)blocks * kMlpWaves);
    k_mlp_rows<true, S><<<blocks, 64 * kMlpWaves, 0, st>>>(net.p.as<float>(), net.F, dX, dt, B, ys, part, sq);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const unsigned sb = (unsigned)((np + 63) / 64);
    if (step) {
        net.step += 1;
        const float c1 = 1.f - std::pow(net.b1, (float)net.step);
        const float c2 = 1.f - std::pow(net.b2, (float)net.step);
        k_mlp_sum<true><<<sb, 256, 0, st>>>(part, parts, np, dg, net.p.as<float>(), net.m.as<float>(),
                                            net.v.as<float>(), net.lr, net.b1, net.b2, net.eps, c1, c2);
    } else {
        k_mlp_sum<false><<<sb, 256, 0, st>>>(part, parts, np, dg, nullptr, nullptr, nullptr, 0.f, 0.f, 0.f, 0.f, 0.f,
                                             0.f);
    }
    return hipGetLastError();
}

static double sum_of(const float *h, int64_t n) {
    double acc = 0;
    for (int64_t i = 0; i < n; ++i) acc += h[i];
    return acc;
}

hipError_t mlp_grad_device(Mlp &net, const float *dX, const float *dt, int64_t B, float *dg, float *loss,
                           hipStream_t st) {
    DevBuf sq;
    hipError_t e;
    if ((e = sq.alloc(sizeof(float) * B)) != hipSuccess) return e;
    std::vector<float> h(B);
    e = grad_launch(net, dX, dt, B, dg, sq.as<float>(), false, st);
    if (e == hipSuccess) e = hipMemcpyAsync(h.data(), sq.p, sizeof(float) * B, hipMemcpyDeviceToHost, st);
    const hipError_t w = hipStreamSynchronize(st);
    if (e == hipSuccess) e = w;
    if (e != hipSuccess) return e;
    if (loss) *loss = (float)(sum_of(h.data(), B) / (double)B);
    return hipSuccess;
}

hipError_t mlp_train_device(Mlp &net, const float *dX, const float *dt, int64_t B, int32_t epochs, int32_t batch,
                            float *losses, hipStream_t st) {
    hipError_t e;
    DevBuf sq;
    if ((e = sq.alloc(sizeof(float) * B)) != hipSuccess) return e;
    std::vector<float> h(losses ? B : 0);
    for (int32_t ep = 0; ep < epochs; ++ep) {
        for (int64_t b0 = 0; b0 < B && e == hipSuccess; b0 += batch)
            e = grad_launch(net, dX + b0 * net.F, dt + b0, std::min<int64_t>(batch, B - b0), net.g.as<float>(),
                            sq.as<float>() + b0, true, st);
        // the epoch's squared errors in one copy (the steps do not wait for it)
        if (e == hipSuccess && losses)
            e = hipMemcpyAsync(h.data(), sq.p, sizeof(float) * B, hipMemcpyDeviceToHost, st);
        const hipError_t w = losses || ep + 1 == epochs || e != hipSuccess ? hipStreamSynchronize(st) : hipSuccess;
        if (e == hipSuccess) e = w;
        if (e != hipSuccess) return e;
        if (!losses) continue;
        double acc = 0;
        for (int64_t b0 = 0; b0 < B; b0 += batch) {
            const int64_t nb = std::min<int64_t>(batch, B - b0);
            acc += (double)(float)(sum_of(h.data() + b0, nb) / (double)nb) * nb;
        }
        losses[ep] = (float)(acc / (double)B);
    }
    return hipSuccess;
}

hipError_t mlp_adam_device(Mlp &net, const float *dg, hipStream_t st) {
    const int64_t np = n_params_of(net.F);
    net.step += 1;
    const float c1 = 1.f - std::pow(net.b1, (float)net.step);
    const float c2 = 1.f - std::pow(net.b2, (float)net.step);
    k_mlp_adam<<<(unsigned)((np + 255) / 256), 256, 0, st>>>(net.p.as<float>(), dg, net.m.as<float>(),
                                                              net.v.as<float>(), np, net.lr, net.b1, net.b2, net.eps,
                                                              c1, c2);
    return hipGetLastError();
}

// SplitMix64 (Steele, Lea and Flood, "Fast splittable pseudorandom number
// generators", 2014): counter-based, used only for the initial weights.
static uint64_t splitmix64(uint64_t x) {
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}

hipError_t mlp_init(Mlp &net, int F, uint64_t seed) {
    net.F = F;
    net.step = 0;
    const int64_t np = n_params_of(F);
    std::vector<float> h(np, 0.f);
    // uniform(-s, s) with s = sqrt(6 / fan_in) for weights (He-uniform), zero biases
    auto fill = [&](int64_t off, int64_t count, int fan_in) {
        const double s = std::sqrt(6.0 / fan_in);
        for (int64_t i = 0; i < count; ++i) {
            const double u = (double)(splitmix64(seed * 0x100000001B3ull + (uint64_t)(off + i)) >> 11) * 0x1.0p-53;
            h[off + i] = (float)((2.0 * u - 1.0) * s);
        }
    };
    fill(0, (int64_t)F * kH, F);
    fill((int64_t)F * kH + kH, kH * kH, kH);
    fill((int64_t)F * kH + kH + kH * kH + kH, kH, kH);
    hipError_t e;
    if ((e = net.p.alloc(sizeof(float) * np)) != hipSuccess) return e;
    if ((e = net.m.alloc(sizeof(float) * np)) != hipSuccess) return e;
    if ((e = net.v.alloc(sizeof(float) * np)) != hipSuccess) return e;
    if ((e = net.g.alloc(sizeof(float) * np)) != hipSuccess) return e;
    if ((e = hipMemcpy(net.p.p, h.data(), sizeof(float) * np, hipMemcpyHostToDevice)) != hipSuccess) return e;
    if ((e = hipMemset(net.m.p, 0, sizeof(float) * np)) != hipSuccess) return e;
    if ((e = hipMemset(net.v.p, 0, sizeof(float) * np)) != hipSuccess) return e;
    net.norm.reset();
    const std::vector<float> zero(F, 0.f), one(F, 1.f);
    return mlp_set_scaling(net, zero.data(), one.data(), 0.f, 1.f);
}

}  // namespace epi
