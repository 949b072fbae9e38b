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
//   forward pass and, when training, the back-propagated terms of every sample
//   (dz1, dz2, dy) beside its activations.
// k_mlp_reduce: one wave per 64 parameters: their gradients, each summed over the
//   batch in sample order, and, in a training step, Adam step k.
// k_mlp_adam:   one thread per parameter; Adam step k with a given gradient.
// k_standardize, k_affine_base: the cost model's input and output scaling
//   around the network, (x - mu) * isd per feature and y * sd + mu, plus the
//   raw base feature (the network predicts the correction to it).
#include <algorithm>
#include <cmath>
#include <vector>

#include "epi_internal.h"

namespace epi {

namespace {

constexpr int kH = kMlpHidden;

__host__ __device__ inline int64_t n_params_of(int F) { return (int64_t)F * kH + kH + kH * kH + kH + kH + 1; }

// What bounds a training step is latency: 512 samples are 9 million multiply-adds,
// nothing for the chip, in a chain of forward, backward, gradient and update.  One
// thread a sample with all weights broadcast from LDS (79 us), then one thread a
// parameter with a load to wait for at each of 512 samples (134 us), then the loss
// fetched by the host took 262 us a step; a wave a tile spreads the batch over 128
// waves, and the sums over the batch keep 192 samples' loads in flight (an epoch of 16 steps of
// 512 and 50k predictions, host copies included: 4.2 -> 0.67 ms).
//
// Every sum is one chain of FP32 fused multiply-adds in a fixed order: over the inputs,
// over the units, over the samples.  Adam divides a gradient by its own size, and a
// ReLU decides on the sign of a sum, so another order (or other bits: FP64 sums moved
// the parameters of some sample sets by up to the learning rate) is another training
// run: the order is part of what the calls return.
constexpr int kMlpWaves = 4;     // waves per workgroup, sharing the staged W2
constexpr int kRow = kH + 1;     // W2's row in LDS: rows and columns free of bank conflicts
constexpr int kRowT = kH + 4;    // h2's row in LDS (16-byte aligned)

// What a training step keeps of every sample, for the sums over the batch:
// activations and terms, a tile of 4 samples after the other, [tile][64] of 4 each (a
// lane of the sums loads its unit's 4 samples at once: a wave has at most 63 loads in
// flight), [B] dy (room for whole tiles) and squared errors.
constexpr int kTileS = 4;
struct MlpRows {
    float4 *h1, *dz1, *dz2, *h2;
    float *dy, *sqerr;
};

// y[s] for every sample; TRAIN also its terms of the gradient of the loss over B
// samples.  S samples a tile.
template <bool TRAIN, int S>
__global__ __launch_bounds__(64 * kMlpWaves) void k_mlp_rows(const float *__restrict__ p, int F,
                                                             const float *__restrict__ X, const float *__restrict__ t,
                                                             int64_t B, float *__restrict__ y, MlpRows rows) {
    __shared__ float W2[kH * kRow];
    __shared__ __align__(16) float W1s[kH * kH];  // W1, for up to 64 inputs
    __shared__ __align__(16) float w3s[kH];
    __shared__ __align__(16) float xb[kMlpWaves][kH][S];      // 64 inputs of the tile's samples
    __shared__ __align__(16) float hb[kMlpWaves][kH][S];      // h1, then dz2
    __shared__ __align__(16) float tb[kMlpWaves][S][kRowT];   // h2
    const int j = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const float *W1 = p, *b1 = p + (int64_t)F * kH, *pW2 = b1 + kH, *b2 = pW2 + kH * kH, *w3 = b2 + kH, *b3 = w3 + kH;
    float(*x)[S] = xb[wv], (*h)[S] = hb[wv], (*h2)[kRowT] = tb[wv];
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
        if (wv == 0) w3s[j] = vw3;
    }
    __syncthreads();  // (the only barrier: from here on the waves work alone)
    auto lds_order = [] {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    const int64_t wave = (int64_t)blockIdx.x * kMlpWaves + wv, waves = (int64_t)gridDim.x * kMlpWaves;
    for (int64_t s0 = wave * S; s0 < B; s0 += waves * S) {
        const int ns = B - s0 < S ? (int)(B - s0) : S;
        float h1[S], z2[S];
#pragma unroll
        for (int q = 0; q < S; ++q) h1[q] = vb1;
        for (int f0 = 0; f0 < F; f0 += kH) {
            // inputs f0 .. f0+63 of the tile (zero for the samples past the batch)
            __builtin_amdgcn_wave_barrier();
            float v[S];
            const int fi = f0 + j < F ? f0 + j : F - 1;
#pragma unroll
            for (int q = 0; q < S; ++q) v[q] = X[(s0 + (q < ns ? q : 0)) * F + fi];
#pragma unroll
            for (int q = 0; q < S; ++q) x[j][q] = q < ns && f0 + j < F ? v[q] : 0.f;
            lds_order();
            const int nf = F - f0 < kH ? F - f0 : kH;
            auto column = [&](const float *w1) {
#pragma unroll 8
                for (int f = 0; f < nf; ++f) {
                    const float wt = w1[f * kH + j];
#pragma unroll
                    for (int q = 0; q < S; ++q) h1[q] = fmaf(x[f][q], wt, h1[q]);
                }
            };
            if (staged) column(W1s);
            else column(W1 + (int64_t)f0 * kH);
        }
#pragma unroll
        for (int q = 0; q < S; ++q) {
            h1[q] = h1[q] > 0.f ? h1[q] : 0.f;  // z1 > 0 <=> h1 > 0
            h[j][q] = h1[q];
            z2[q] = vb2;
        }
        lds_order();
#pragma unroll 8
        for (int a = 0; a < kH; ++a) {
            const float wt = W2[a * kRow + j];
#pragma unroll
            for (int q = 0; q < S; ++q) z2[q] = fmaf(h[a][q], wt, z2[q]);
        }
        // the output is one chain over the units: a lane per sample takes it
#pragma unroll
        for (int q = 0; q < S; ++q) h2[q][j] = z2[q] > 0.f ? z2[q] : 0.f;
        lds_order();
        float out = vb3;
        const int mine = j % S;
#pragma unroll 4
        for (int a = 0; a < kH; a += 4) {
            const float4 u = *reinterpret_cast<const float4 *>(&h2[mine][a]);
            const float4 w = *reinterpret_cast<const float4 *>(&w3s[a]);
            out = fmaf(u.x, w.x, out);
            out = fmaf(u.y, w.y, out);
            out = fmaf(u.z, w.z, out);
            out = fmaf(u.w, w.w, out);
        }
        if (j < ns) y[s0 + j] = out;
        if constexpr (TRAIN) {
            // dz2 = dy * w3 * [z2 > 0];  dz1 = (dz2 W2^T) * [z1 > 0]
            const float r = mine < ns ? out - t[s0 + mine] : 0.f;
            const float dy1 = 2.f * r / (float)B;
            if (j < ns) {
                rows.sqerr[s0 + j] = r * r;
                rows.dy[s0 + j] = dy1;
            }
            static_assert(!TRAIN || S == kTileS, "a tile's samples are kept together");
            float dz1[S], dz2[S];
#pragma unroll
            for (int q = 0; q < S; ++q) {
                const float dy = __shfl(dy1, q, 64);
                dz2[q] = z2[q] > 0.f ? dy * vw3 : 0.f;
                z2[q] = z2[q] > 0.f ? z2[q] : 0.f;  // now h2
                h[j][q] = dz2[q];
                dz1[q] = 0.f;
            }
            const int64_t o = s0 / S * kH + j;
            rows.h1[o] = make_float4(h1[0], h1[1], h1[2], h1[3]);
            rows.h2[o] = make_float4(z2[0], z2[1], z2[2], z2[3]);
            rows.dz2[o] = make_float4(dz2[0], dz2[1], dz2[2], dz2[3]);
            lds_order();
#pragma unroll 8
            for (int k = 0; k < kH; ++k) {  // lane j = unit j of the first layer
                const float wt = W2[j * kRow + k];
#pragma unroll
                for (int q = 0; q < S; ++q) dz1[q] = fmaf(h[k][q], wt, dz1[q]);
            }
#pragma unroll
            for (int q = 0; q < S; ++q) dz1[q] = h1[q] > 0.f ? dz1[q] : 0.f;
            rows.dz1[o] = make_float4(dz1[0], dz1[1], dz1[2], dz1[3]);
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// (every product that is added is a fused multiply-add, whatever the kernel)
__device__ __forceinline__ void adam(float *__restrict__ p, float *__restrict__ m, float *__restrict__ v, int64_t q,
                                     float gq, float lr, float b1, float b2, float eps, float c1, float c2) {
#pragma clang fp contract(off)
    const float mq = fmaf(1.f - b1, gq, b1 * m[q]);
    const float vq = fmaf((1.f - b2) * gq, gq, b2 * v[q]);
    m[q] = mq;
    v[q] = vq;
    p[q] = p[q] - lr * (mq / c1) / (sqrtf(vq / c2) + eps);
}

// Gradients of parameters 64 row .. 64 row + 63, each the chain acc = u_i v_i + acc
// over the samples i in order (a bias: u = 1); ADAM: and the step with them.
// Lane j: parameter j of the row.  u is the same for all lanes (the last row, the
// output's bias, has one parameter).  Chunks of 64 samples: the loads of the next two
// are in flight under one's chain (what was written a launch before comes from beyond
// L2, some 2 us away).
template <bool ADAM>
__global__ __launch_bounds__(64) void k_mlp_reduce(int F, const float *__restrict__ X, int64_t B, MlpRows rows,
                                                   float *__restrict__ g, float *__restrict__ p,
                                                   float *__restrict__ m, float *__restrict__ v, float lr, float b1,
                                                   float b2, float eps, float c1, float c2) {
    const int row = blockIdx.x, j = threadIdx.x;
    constexpr int kTiles = kH / kTileS;  // of a chunk
    // u of sample i: u[i * us], or of a unit's activations (us = 0); e of tile i: e[i * et]
    const float *u = nullptr;
    const float4 *e = rows.dz1 + j;
    int64_t us = 0, et = kH;
    int r = row;
    if (r < F) {  // W1[f][j]: x_f dz1_j
        u = X + r;
        us = F;
    } else if ((r -= F) == 0) {  // b1
    } else if ((r -= 1) < kH) {  // W2[a][j]: h1_a dz2_j
        u = reinterpret_cast<const float *>(rows.h1 + r);
        e = rows.dz2 + j;
    } else if ((r -= kH) == 0) {  // b2
        e = rows.dz2 + j;
    } else if (r == 1) {  // w3[j]: h2_j dy
        u = rows.dy;
        us = 1;
        e = rows.h2 + j;
    } else {  // b3
        e = reinterpret_cast<const float4 *>(rows.dy);
        et = 1;
    }
    struct Chunk {
        float4 e[kTiles];
        float u;
    };
    const int64_t last = B - 1, last_tile = last / kTileS;
    auto load = [&](Chunk &c, int64_t i0) __attribute__((always_inline)) {
        if (i0 >= B) return;  // uniform
        const int64_t i = i0 + j < last ? i0 + j : last;
        c.u = u ? u[us ? i * us : i / kTileS * kH * kTileS + i % kTileS] : 1.f;
#pragma unroll
        for (int k = 0; k < kTiles; ++k) {
            const int64_t t = i0 / kTileS + k < last_tile ? i0 / kTileS + k : last_tile;
            c.e[k] = e[t * et];
        }
    };
    float acc = 0.f;
    auto chain = [&](const Chunk &c, int64_t i0) __attribute__((always_inline)) {
        auto term = [&](int k) __attribute__((always_inline)) {
            const float uk = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(c.u), k));
            const float4 &q = c.e[k / kTileS];
            acc = fmaf(uk, k % kTileS == 0 ? q.x : k % kTileS == 1 ? q.y : k % kTileS == 2 ? q.z : q.w, acc);
        };
        if (B - i0 >= kH) {  // uniform
#pragma unroll
            for (int k = 0; k < kH; ++k) term(k);
        } else {
            const int n = (int)(B - i0);
#pragma unroll
            for (int k = 0; k < kH; ++k)
                if (k < n) term(k);  // uniform
        }
    };
    Chunk ca, cb, cc;
    load(ca, 0);
    load(cb, kH);
    load(cc, 2 * kH);
    for (int64_t i0 = 0; i0 < B; i0 += 3 * kH) {
        chain(ca, i0);
        load(ca, i0 + 3 * kH);
        if (i0 + kH >= B) break;
        chain(cb, i0 + kH);
        load(cb, i0 + 4 * kH);
        if (i0 + 2 * kH >= B) break;
        chain(cc, i0 + 2 * kH);
        load(cc, i0 + 5 * kH);
    }
    const int64_t q = (int64_t)row * kH + j;
    if (q >= n_params_of(F)) return;
    g[q] = acc;
    if constexpr (ADAM) adam(p, m, v, q, acc, lr, b1, b2, eps, c1, c2);
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
        net.p.as<float>(), net.F, dX, nullptr, B, dy, MlpRows{});
    return hipGetLastError();
}

// Gradient over B device samples into dg, the squared errors into sq (device);
// step: then the Adam step with it.
static hipError_t grad_launch(Mlp &net, const float *dX, const float *dt, int64_t B, float *dg, float *sq, bool step,
                              hipStream_t st) {
    hipError_t e;
    if (!mlp_fits(net)) return hipErrorInvalidValue;
    constexpr int S = kTileS;
    const int64_t np = n_params_of(net.F), tiles = (B + S - 1) / S;
    const size_t need = sizeof(float) * (size_t)tiles * S * (4 * kH + 2);
    if (net.act.bytes < need) {
        if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
        if ((e = net.act.alloc(need)) != hipSuccess) return e;
    }
    const size_t w = (size_t)tiles * kH;
    float4 *base = net.act.as<float4>();
    MlpRows rows{base, base + w, base + 2 * w, base + 3 * w, reinterpret_cast<float *>(base + 4 * w), sq};
    float *ys = rows.dy + tiles * S;
    const int64_t blocks = (tiles + kMlpWaves - 1) / kMlpWaves;
    k_mlp_rows<true, S><<<(unsigned)std::min<int64_t>(blocks, 1024), 64 * kMlpWaves, 0, st>>>(
        net.p.as<float>(), net.F, dX, dt, B, ys, rows);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const unsigned nr = (unsigned)((np + kH - 1) / kH);
    if (step) {
        net.step += 1;
        const float c1 = 1.f - std::pow(net.b1, (float)net.step);
        const float c2 = 1.f - std::pow(net.b2, (float)net.step);
        k_mlp_reduce<true><<<nr, kH, 0, st>>>(net.F, dX, B, rows, dg, net.p.as<float>(), net.m.as<float>(),
                                              net.v.as<float>(), net.lr, net.b1, net.b2, net.eps, c1, c2);
    } else {
        k_mlp_reduce<false><<<nr, kH, 0, st>>>(net.F, dX, B, rows, dg, nullptr, nullptr, nullptr, 0.f, 0.f, 0.f, 0.f,
                                               0.f, 0.f);
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
