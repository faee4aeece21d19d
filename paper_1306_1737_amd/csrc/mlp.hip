// Learned Verlet-buffer predictor: hand-written training and inference
// kernels for an 8-64-64-1 multilayer perceptron (not part of the paper; it
// learns the buffer the paper's drift criterion needs, Sec. 5, from exact
// missed-pair recounts).
//
// x (8 raw features) -> normalised to [-1, 1] with the model's feature ranges
//   -> h1 = tanh(W1 x + b1) -> h2 = tanh(W2 h1 + b2) -> y = softplus(w3.h2 + b3)
// Loss: mean squared error over the batch; optimiser: Adam with bias
// correction (beta1 0.9, beta2 0.999, eps 1e-8).  Flat parameter order:
// W1 (64x8 row-major), b1, W2 (64x64 row-major), b2, w3, b3 -- 4801 floats.
//
// Mapping: a workgroup of four wavefronts; lane j of a wavefront is hidden
// unit j of both layers and keeps its rows of W1 and W2 (and their gradient
// accumulators) in registers.  Hidden activations and the layer-2 deltas are
// broadcast through LDS; the column access W2^T delta2 reads a padded LDS
// copy of W2 without bank conflicts.
//
// A sample is a chain of about 2 us on one wavefront (LDS round trips, tanh,
// the output sum), so a minibatch on one workgroup is bound by that chain
// times batch / 4.  The batch is therefore spread over up to kMlpParts
// workgroups, each writing the gradient of its share to scratch; a second
// launch sums the shares in a fixed order and applies Adam (256 samples: 144
// us a call on one workgroup, 13.3 us on 64).
#include "internal.h"

namespace {

constexpr int NF = 8, NH = 64;
constexpr int OFF_W1 = 0, OFF_B1 = NH * NF, OFF_W2 = OFF_B1 + NH, OFF_B2 = OFF_W2 + NH * NH, OFF_W3 = OFF_B2 + NH,
              OFF_B3 = OFF_W3 + NH, NPARAM = OFF_B3 + 1;
static_assert(NPARAM == 4801, "parameter count");
constexpr int kMlpParts = 128;                          // most workgroups a batch is spread over
constexpr int kMlpRow = (NPARAM + 1 + 63) / 64 * 64;    // floats per gradient row: parameters, then the loss sum


struct MlpArgs {
    float *params, *m, *v;
    int *step;
    const float *lo, *hi;
    const float *X, *y;
    int batch;
    float lr;
    float *loss;
    float *grad_out;   // non-null: write the batch gradient, do not update
    float *parts;      // gradient rows of the workgroups (kMlpRow floats each)
    float *y_out;      // inference output
};

__device__ inline void wave_sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline float wsum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ inline float softplus(float z) { return fmaxf(z, 0.0f) + log1pf(expf(-fabsf(z))); }

__device__ inline float sigmoid(float z) { return 1.0f / (1.0f + expf(-z)); }

constexpr int GROW = NH + 1;   // padded W2 gradient rows in LDS: lane j's element i lies in bank (j + i) mod 32
// LDS address of flat parameter p (the W2 block padded), and of the loss sum after the last parameter
__device__ inline int gaddr(int p) {
    return p < OFF_W2 ? p : (p < OFF_B2 ? OFF_W2 + (p - OFF_W2) / NH * GROW + (p - OFF_W2) % NH : p + NH);
}

__device__ inline void adam(const MlpArgs &a, int i, float g, int t) {
    const float c1 = 1.0f / (1.0f - powf(0.9f, (float)t)), c2 = 1.0f / (1.0f - powf(0.999f, (float)t));
    const float m = 0.9f * a.m[i] + 0.1f * g;
    const float v = 0.999f * a.v[i] + 0.001f * g * g;
    a.m[i] = m;
    a.v[i] = v;
    a.params[i] -= a.lr * (m * c1) / (sqrtf(v * c2) + 1e-8f);
}

// Gradient of the samples s = wave, wave + waves, ... of this workgroup.
// PARTS: the sums go to this workgroup's row of a.parts (k_mlp_finish adds
// the rows); otherwise one workgroup holds the whole batch and finishes it.
template <bool PARTS>
__global__ __launch_bounds__(256) void k_mlp_step(MlpArgs a) {
    __shared__ float w2s[NH * (NH + 1)];
    __shared__ float h1s[4][NH], d2s[4][NH];
    __shared__ float gacc[NPARAM + 1 + NH];   // gradient (gaddr order), then the loss sum
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    for (int i = tid; i < NH * NH; i += 256) w2s[(i / NH) * (NH + 1) + i % NH] = a.params[OFF_W2 + i];
    __syncthreads();
    float w1[NF], gw1[NF], w2[NH], gw2[NH], lo[NF], sc[NF];
#pragma unroll
    for (int i = 0; i < NF; ++i) {
        w1[i] = a.params[OFF_W1 + lane * NF + i];
        gw1[i] = 0.0f;
        lo[i] = a.lo[i];
        sc[i] = 2.0f / (a.hi[i] - a.lo[i]);
    }
#pragma unroll
    for (int i = 0; i < NH; ++i) {
        w2[i] = w2s[lane * (NH + 1) + i];
        gw2[i] = 0.0f;
    }
    const float b1 = a.params[OFF_B1 + lane], b2 = a.params[OFF_B2 + lane], w3 = a.params[OFF_W3 + lane];
    const float b3 = a.params[OFF_B3];
    float gb1 = 0.0f, gb2 = 0.0f, gw3 = 0.0f, gb3 = 0.0f, lsum = 0.0f;
    const float inv_b = 2.0f / (float)a.batch;
    for (int s = blockIdx.x * 4 + w; s < a.batch; s += gridDim.x * 4) {
        float x[NF];
#pragma unroll
        for (int i = 0; i < NF; ++i) x[i] = (a.X[s * NF + i] - lo[i]) * sc[i] - 1.0f;
        float z1 = b1;
#pragma unroll
        for (int i = 0; i < NF; ++i) z1 = fmaf(w1[i], x[i], z1);
        const float h1 = tanhf(z1);
        h1s[w][lane] = h1;
        wave_sync_lds();
        float z2 = b2;
#pragma unroll
        for (int i = 0; i < NH; ++i) z2 = fmaf(w2[i], h1s[w][i], z2);
        const float h2 = tanhf(z2);
        const float z3 = wsum(w3 * h2) + b3;
        const float r = softplus(z3) - a.y[s];
        lsum += r * r;
        const float d3 = inv_b * r * sigmoid(z3);
        gw3 = fmaf(d3, h2, gw3);
        gb3 += d3;
        const float d2 = d3 * w3 * (1.0f - h2 * h2);
        gb2 += d2;
#pragma unroll
        for (int i = 0; i < NH; ++i) gw2[i] = fmaf(d2, h1s[w][i], gw2[i]);
        d2s[w][lane] = d2;
        wave_sync_lds();
        float s1 = 0.0f;
#pragma unroll 16
        for (int k = 0; k < NH; ++k) s1 = fmaf(w2s[k * (NH + 1) + lane], d2s[w][k], s1);
        const float d1 = (1.0f - h1 * h1) * s1;
        gb1 += d1;
#pragma unroll
        for (int i = 0; i < NF; ++i) gw1[i] = fmaf(d1, x[i], gw1[i]);
        wave_sync_lds();   // before the next sample overwrites h1s / d2s
    }
    // the four wavefronts' sums, added in wavefront order
    for (int k = 0; k < 4; ++k) {
        if (w == k) {
            auto put = [&](int at, float v) { gacc[at] = k == 0 ? v : gacc[at] + v; };
#pragma unroll
            for (int i = 0; i < NF; ++i) put(OFF_W1 + lane * NF + i, gw1[i]);
            put(OFF_B1 + lane, gb1);
#pragma unroll
            for (int i = 0; i < NH; ++i) put(OFF_W2 + lane * GROW + i, gw2[i]);
            put(gaddr(OFF_B2) + lane, gb2);
            put(gaddr(OFF_W3) + lane, gw3);
            if (lane == 0) {
                put(gaddr(OFF_B3), gb3);
                put(gaddr(NPARAM), lsum);
            }
        }
        __syncthreads();
    }
    if constexpr (PARTS) {
        float *row = a.parts + (size_t)blockIdx.x * kMlpRow;
        for (int i = tid; i <= NPARAM; i += 256) row[i] = gacc[gaddr(i)];
        if (!a.grad_out && blockIdx.x == 0 && tid == 0) *a.step += 1;   // read by k_mlp_finish
    } else {
        if (a.loss && tid == 0) *a.loss = gacc[gaddr(NPARAM)] / (float)a.batch;
        const int t = *a.step + 1;
        for (int i = tid; i < NPARAM; i += 256) {
            if (a.grad_out) a.grad_out[i] = gacc[gaddr(i)];
            else adam(a, i, gacc[gaddr(i)], t);
        }
        __syncthreads();
        if (!a.grad_out && tid == 0) *a.step = t;
    }
}

// Sum of the workgroups' gradient rows (64 parameters per workgroup; each of its wavefronts adds every
// fourth row, the four sums are added in order), then Adam or the gradient output; the loss is value NPARAM.
// Summed in FP64, which costs no time here (the launch waits for the rows' loads) and rounds each value once.
__global__ __launch_bounds__(256) void k_mlp_finish(MlpArgs a, int nparts) {
    __shared__ double red[4][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, i = blockIdx.x * 64 + lane;
    double s = 0.0;
    if (i <= NPARAM) {
#pragma unroll 8
        for (int k = w; k < nparts; k += 4) s += a.parts[(size_t)k * kMlpRow + i];
    }
    red[w][lane] = s;
    __syncthreads();
    if (w > 0 || i > NPARAM) return;
    const float g = (float)(((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane]);
    if (i == NPARAM) {
        if (a.loss) *a.loss = g / (float)a.batch;
    } else if (a.grad_out) {
        a.grad_out[i] = g;
    } else {
        adam(a, i, g, *a.step);
    }
}

// Inference: each wavefront evaluates samples s = wave, wave + waves, ...
__global__ __launch_bounds__(256) void k_mlp_infer(MlpArgs a) {
    __shared__ float h1s[4][NH];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    float w1[NF], w2[NH], lo[NF], sc[NF];
#pragma unroll
    for (int i = 0; i < NF; ++i) {
        w1[i] = a.params[OFF_W1 + lane * NF + i];
        lo[i] = a.lo[i];
        sc[i] = 2.0f / (a.hi[i] - a.lo[i]);
    }
#pragma unroll
    for (int i = 0; i < NH; ++i) w2[i] = a.params[OFF_W2 + lane * NH + i];
    const float b1 = a.params[OFF_B1 + lane], b2 = a.params[OFF_B2 + lane], w3 = a.params[OFF_W3 + lane];
    const float b3 = a.params[OFF_B3];
    for (int s = blockIdx.x * 4 + w; s < a.batch; s += gridDim.x * 4) {
        float z1 = b1;
#pragma unroll
        for (int i = 0; i < NF; ++i) z1 = fmaf(w1[i], (a.X[s * NF + i] - lo[i]) * sc[i] - 1.0f, z1);
        h1s[w][lane] = tanhf(z1);
        wave_sync_lds();
        float z2 = b2;
#pragma unroll
        for (int i = 0; i < NH; ++i) z2 = fmaf(w2[i], h1s[w][i], z2);
        const float z3 = wsum(w3 * tanhf(z2)) + b3;
        if (lane == 0) a.y_out[s] = softplus(z3);
        wave_sync_lds();
    }
}

}  // namespace

namespace mxn {

int launch_mlp_step(nb_ctx *ctx, nb_mlp *mlp, const float *X, const float *y, int batch, float lr, float *loss,
                    float *grad_out) {
    MlpArgs a{};
    a.params = (float *)mlp->params.p;
    a.m = (float *)mlp->m.p;
    a.v = (float *)mlp->v.p;
    a.step = (int *)mlp->step.p;
    a.lo = (const float *)mlp->lo.p;
    a.hi = (const float *)mlp->hi.p;
    a.X = X;
    a.y = y;
    a.batch = batch;
    a.lr = lr;
    a.loss = loss;
    a.grad_out = grad_out;
    // Two samples per wavefront or fewer: the second launch costs more than the chains it shortens.
    const int nparts = batch <= 8 ? 1 : std::min((batch + 3) / 4, kMlpParts);
    std::lock_guard<std::mutex> lock(mlp->scratch.mu);
    if (nparts > 1) a.parts = (float *)mlp->scratch.get(ctx, sizeof(float) * kMlpRow * kMlpParts);
    if (!a.parts) {
        k_mlp_step<false><<<1, 256, 0, ctx->stream>>>(a);
    } else {
        k_mlp_step<true><<<nparts, 256, 0, ctx->stream>>>(a);
        k_mlp_finish<<<(NPARAM + 1 + 63) / 64, 256, 0, ctx->stream>>>(a, nparts);
    }
    MXN_HIP(hipGetLastError());
    return NB_OK;
}

int launch_mlp_infer(nb_ctx *ctx, const nb_mlp *mlp, const float *X, int batch, float *y) {
    MlpArgs a{};
    a.params = (float *)mlp->params.p;
    a.lo = (const float *)mlp->lo.p;
    a.hi = (const float *)mlp->hi.p;
    a.X = X;
    a.batch = batch;
    a.y_out = y;
    int nb = (batch + 3) / 4;
    if (nb > 1024) nb = 1024;
    if (nb < 1) nb = 1;
    k_mlp_infer<<<nb, 256, 0, ctx->stream>>>(a);
    MXN_HIP(hipGetLastError());
    return NB_OK;
}

}  // namespace mxn
