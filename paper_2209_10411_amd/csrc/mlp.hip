// Warm-start MLP: link features, batched forward/backward and Adam for
// training (own kernels, FP32 accumulation; one thread per output element,
// fixed-order sums so that every result is deterministic).  The one-link
// inference inside the link solver is in kernels.hip.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "mlp_dev.h"

namespace mdl {

namespace {
__constant__ int m_ex[19] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0};
__constant__ int m_ey[19] = {0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1};
__constant__ int m_ez[19] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1};

size_t al(size_t x) { return (x + 255) & ~size_t(255); }
}  // namespace

// Blob: theta, m, v (FP32 [P]); w16 (FP16 [P]); t; workspace for
// MLP_MAX_BATCH samples.
size_t mlp_blob_bytes() {
    size_t o = 0;
    o = al(o + 4 * (size_t)MLP_P);          // theta
    o = al(o + 4 * (size_t)MLP_P);          // m
    o = al(o + 4 * (size_t)MLP_P);          // v
    o = al(o + 2 * (size_t)MLP_P);          // w16
    o = al(o + 8);                          // t
    o = al(o + 4 * (size_t)MLP_MAX_BATCH * MLP_H);  // h1
    o = al(o + 4 * (size_t)MLP_MAX_BATCH * MLP_H);  // h2
    o = al(o + 4 * (size_t)MLP_MAX_BATCH * MLP_OUT);  // out
    o = al(o + 4 * (size_t)MLP_MAX_BATCH * MLP_OUT);  // dout
    o = al(o + 4 * (size_t)MLP_MAX_BATCH * MLP_H);  // dz1
    o = al(o + 4 * (size_t)MLP_MAX_BATCH * MLP_H);  // dz2
    o = al(o + 4 * (size_t)MLP_P);          // g
    o = al(o + 4);                          // loss
    o = al(o + 4 * (size_t)16 * (MLP_IN + 1) * MLP_H);  // weight-gradient slices
    return o;
}

MlpBlob mlp_blob(void *base) {
    char *b = (char *)base;
    MlpBlob r;
    size_t o = 0;
    auto take = [&](size_t bytes) { char *p = b + o; o = al(o + bytes); return p; };
    r.theta = (float *)take(4 * (size_t)MLP_P);
    r.m = (float *)take(4 * (size_t)MLP_P);
    r.v = (float *)take(4 * (size_t)MLP_P);
    r.w16 = (_Float16 *)take(2 * (size_t)MLP_P);
    r.t = (long long *)take(8);
    r.h1 = (float *)take(4 * (size_t)MLP_MAX_BATCH * MLP_H);
    r.h2 = (float *)take(4 * (size_t)MLP_MAX_BATCH * MLP_H);
    r.out = (float *)take(4 * (size_t)MLP_MAX_BATCH * MLP_OUT);
    take(4 * (size_t)MLP_MAX_BATCH * MLP_OUT);  // unused, like the next but one: the blob keeps its size
    r.sq = (float *)take(4 * (size_t)MLP_MAX_BATCH * MLP_H);
    take(4 * (size_t)MLP_MAX_BATCH * MLP_H);
    r.g = (float *)take(4 * (size_t)MLP_P);
    r.loss = (float *)take(4);
    return r;
}

__global__ void k_mlp_init(float *theta, float *m, float *v, _Float16 *w16, long long *t) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < MLP_P) {
        m[i] = 0.f;
        v[i] = 0.f;
        w16[i] = (_Float16)theta[i];
    }
    if (i == 0) *t = 0;
}

// z = h_prev W + b for sample b, unit n; tanh (stored as TA) or linear (FP32 out)
template <typename TA, typename TW>
__global__ void k_mlp_layer(const TA *__restrict__ X, int K, const TW *__restrict__ W, int offW, int offB, int N,
                            int B, TA *__restrict__ H, float *__restrict__ out) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= B * N) return;
    const int b = idx / N, n = idx - b * N;
    float z = (float)W[offB + n];
    for (int k = 0; k < K; ++k) z += (float)X[(long long)b * K + k] * (float)W[offW + k * N + n];
    if (H) H[idx] = (TA)tanhf(z);
    else out[idx] = z;
}

// fixed-order sum of the squared errors (one block of 256 threads)
__global__ void k_mlp_loss(const float *__restrict__ sq, int n, int B, float *__restrict__ loss) {
    __shared__ float s[256];
    float a = 0.f;
    for (int i = threadIdx.x; i < n; i += 256) a += sq[i];
    s[threadIdx.x] = a;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) s[threadIdx.x] += s[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = s[0] / (float)B;
}

// Forward, loss gradient and backward of one slice of a batch of B samples in
// one block (MLP_SLICES slices, slice s the samples B s / 16 .. B (s + 1) / 16):
// tiles of 16 samples, two per wave, with weights, activations and layer
// gradients in LDS; lane u forms unit u, each sum over its inputs in order (a
// weight is read once for both samples, their inputs as one broadcast).  The slice's share of every parameter's gradient
// (sum_b h[b][k] dZ[b][n], b in order; the bias row h = 1) stays in registers
// over the tiles and goes to part[s][P] in parameter order.  sq (or NULL):
// squared errors of the targeted outputs for the loss.  One launch takes the
// place of a launch per layer and direction (17 a minibatch with the optimiser,
// all of it launches and their latency): minibatches of 256 take 17 us each
// instead of 93, of 4096 160 instead of 340.
constexpr int MLP_SLICES = 16;
constexpr int MLP_T = 16, MLP_TP = 20;  // samples per tile; padded row (16-byte aligned, banks spread)
constexpr int MLP_W = 8, MLP_N = MLP_T / MLP_W;  // waves, samples of a tile per wave
constexpr int MLP_BLK = 64 * MLP_W;
// FULL: every slice holds whole tiles (B a multiple of 256).  Else a wave past
// the slice's end leaves the layers out: batches of 64 take 16.1 us instead of
// 18.2 so, but whole tiles 2 % more than without the branches.
template <typename TA, typename TW, bool FULL>
__global__ __launch_bounds__(MLP_BLK) void k_mlp_slice(const TA *__restrict__ X, const TW *__restrict__ W,
                                                   const float *__restrict__ T, int B, float *__restrict__ part,
                                                   float *__restrict__ sq) {
    constexpr int W2P = MLP_H + 2;  // padded row of W2 (its backward reads a column)
    __shared__ __align__(16) TW w1[MLP_IN * MLP_H], w2[MLP_H * W2P], w3[MLP_H * MLP_OUT], bias[2 * MLP_H + MLP_OUT];
    __shared__ __align__(16) float x[MLP_IN][MLP_TP], h1[MLP_H][MLP_TP], h2[MLP_H][MLP_TP], d1[MLP_H][MLP_TP],
        d2[MLP_H][MLP_TP], d3[MLP_OUT][MLP_TP];
    const int t = threadIdx.x, u = t & 63, w = t >> 6, q0 = MLP_N * w;
    {  // weights, four bytes at a time (both matrices start on a multiple of four)
        constexpr int PW = 4 / sizeof(TW);
#pragma unroll
        for (int i = t * PW; i < MLP_IN * MLP_H; i += MLP_BLK * PW) __builtin_memcpy(&w1[i], &W[MLP_OFF_W1 + i], 4);
#pragma unroll
        for (int i = t * PW; i < MLP_H * MLP_H; i += MLP_BLK * PW)
            __builtin_memcpy(&w2[(i / MLP_H) * W2P + i % MLP_H], &W[MLP_OFF_W2 + i], 4);
    }
    if (t < MLP_H * MLP_OUT) w3[t] = W[MLP_OFF_W3 + t];
    if (t < MLP_H) {
        bias[t] = W[MLP_OFF_B1 + t];
        bias[MLP_H + t] = W[MLP_OFF_B2 + t];
    }
    if (t < MLP_OUT) bias[2 * MLP_H + t] = W[MLP_OFF_B3 + t];
    // row k of a weight gradient belongs to wave k % MLP_W; lane u has column u
    constexpr int R1 = (MLP_IN + 1) / MLP_W, R2 = MLP_H / MLP_W + 1;
    float g1[R1], g2[R2], g3[2] = {0.f, 0.f};  // g3 (t < 256): row t / 4 of W3, column t % 4, and (t < 4) its bias
#pragma unroll
    for (int r = 0; r < R1; ++r) g1[r] = 0.f;
#pragma unroll
    for (int r = 0; r < R2; ++r) g2[r] = 0.f;
    const int s = blockIdx.x;
    const int b0 = (int)((long long)B * s / MLP_SLICES), b1 = (int)((long long)B * (s + 1) / MLP_SLICES);
    for (int base = b0; base < b1; base += MLP_T) {
        // Samples past the slice's end have no output gradient, but with a weight that
        // FP16 holds as infinite the activations of zeros are NaN, and so is their
        // product with a zero gradient: a wave past the end has activations and layer
        // gradients of zero, one that reaches past it takes the last sample again.
        const int nb = FULL ? MLP_T : min(MLP_T, b1 - base), filled = (nb + MLP_N - 1) / MLP_N * MLP_N;
        const bool live = FULL || __builtin_amdgcn_readfirstlane(q0) < nb;
        if (base > b0) __syncthreads();  // the last tile's arrays are read
#pragma unroll
        for (int i = t; i < MLP_T * MLP_IN; i += MLP_BLK) {
            const int b = i / MLP_IN, k = i - b * MLP_IN;
            x[k][b] = b < filled ? (float)X[(long long)(base + min(b, nb - 1)) * MLP_IN + k] : 0.f;
        }
        __syncthreads();
        typedef float vec __attribute__((ext_vector_type(MLP_N)));
        auto layer = [&](const float(*in)[MLP_TP], int K, const TW *wt, int stride, float zb, float z[MLP_N]) {
#pragma unroll
            for (int q = 0; q < MLP_N; ++q) z[q] = zb;
#pragma unroll 16
            for (int k = 0; k < K; ++k) {
                const vec v = *(const vec *)&in[k][q0];
                const float wk = (float)wt[k * stride + u];
#pragma unroll
                for (int q = 0; q < MLP_N; ++q) z[q] += v[q] * wk;
            }
        };
        auto none = [&](float(*a)[MLP_TP]) {
#pragma unroll
            for (int q = 0; q < MLP_N; ++q) a[u][q0 + q] = 0.f;
        };
        float z[MLP_N];
        if (live) {
            layer(x, MLP_IN, w1, MLP_H, (float)bias[u], z);
#pragma unroll
            for (int q = 0; q < MLP_N; ++q) h1[u][q0 + q] = (float)(TA)tanhf(z[q]);
        } else {
            none(h1);
        }
        __syncthreads();
        if (live) {
            layer(h1, MLP_H, w2, W2P, (float)bias[MLP_H + u], z);
#pragma unroll
            for (int q = 0; q < MLP_N; ++q) h2[u][q0 + q] = (float)(TA)tanhf(z[q]);
        } else {
            none(h2);
        }
        __syncthreads();
        if (t < MLP_T * MLP_OUT) {  // outputs and the masked squared error's gradient (mean over the batch)
            const int b = t / MLP_OUT, j = t - b * MLP_OUT;
            float o = (float)bias[2 * MLP_H + j];
#pragma unroll 16
            for (int k = 0; k < MLP_H; ++k) o += h2[k][b] * (float)w3[k * MLP_OUT + j];
            const bool task = x[6][b] > 0.5f, on = (task ? j > 0 : j == 0) && b < nb;
            const long long at = (long long)(base + (b < nb ? b : 0)) * MLP_OUT + j;
            const float d = o - T[at];
            d3[j][b] = on ? 2.f * d / (float)B : 0.f;
            if (sq && b < nb) sq[at] = on ? d * d : 0.f;
        }
        __syncthreads();
        if (live) {
#pragma unroll
            for (int q = 0; q < MLP_N; ++q) {
                float e = 0.f;
#pragma unroll
                for (int n = 0; n < MLP_OUT; ++n) e += d3[n][q0 + q] * (float)w3[u * MLP_OUT + n];
                const float h = h2[u][q0 + q];
                d2[u][q0 + q] = e * (1.f - h * h);
            }
        } else {
            none(d2);
        }
        __syncthreads();
        if (live) {
            float e[MLP_N] = {};
#pragma unroll 16
            for (int n = 0; n < MLP_H; ++n) {
                const vec v = *(const vec *)&d2[n][q0];
                const float wn = (float)w2[u * W2P + n];
#pragma unroll
                for (int q = 0; q < MLP_N; ++q) e[q] += v[q] * wn;
            }
#pragma unroll
            for (int q = 0; q < MLP_N; ++q) {
                const float h = h1[u][q0 + q];
                d1[u][q0 + q] = e[q] * (1.f - h * h);
            }
        } else {
            none(d1);
        }
        __syncthreads();
        // gradients: samples past the slice's end have zero layer gradients
        auto rows = [&](const float(*in)[MLP_TP], int K, const float(*dz)[MLP_TP], float *g, int R) {
            float dv[MLP_T];
#pragma unroll
            for (int b = 0; b < MLP_T; ++b) dv[b] = dz[u][b];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int k = MLP_W * r + w;
                if (k > K) continue;  // wave-uniform
                float v = g[r];
#pragma unroll
                for (int b = 0; b < MLP_T; ++b) v += (k < K ? in[k][b] : 1.f) * dv[b];
                g[r] = v;
                if (r & 1) __builtin_amdgcn_sched_barrier(0);  // two rows' inputs at a time in registers
            }
        };
        rows(x, MLP_IN, d1, g1, R1);
        rows(h1, MLP_H, d2, g2, R2);
        if (t < MLP_H * MLP_OUT)
            for (int b = 0; b < nb; ++b) {
                g3[0] += h2[t / MLP_OUT][b] * d3[t % MLP_OUT][b];
                if (t < MLP_OUT) g3[1] += d3[t][b];
            }
    }
    float *g = part + (long long)s * MLP_P;
#pragma unroll
    for (int r = 0; r < R1; ++r) {
        const int k = MLP_W * r + w;  // k = MLP_IN: the bias row follows the weights
        if (k <= MLP_IN) g[MLP_OFF_W1 + k * MLP_H + u] = g1[r];
    }
#pragma unroll
    for (int r = 0; r < R2; ++r) {
        const int k = MLP_W * r + w;
        if (k <= MLP_H) g[MLP_OFF_W2 + k * MLP_H + u] = g2[r];
    }
    if (t < MLP_H * MLP_OUT) g[MLP_OFF_W3 + t] = g3[0];
    if (t < MLP_OUT) g[MLP_OFF_B3 + t] = g3[1];
}
static_assert(MLP_OFF_B1 == MLP_OFF_W1 + MLP_IN * MLP_H && MLP_OFF_B2 == MLP_OFF_W2 + MLP_H * MLP_H &&
                  MLP_H * MLP_OUT <= MLP_BLK && (MLP_IN + 1) % MLP_W == 0 && MLP_H % MLP_W == 0,
              "k_mlp_slice's layout");

// g = the slices' shares in order.
__device__ __forceinline__ float mlp_grad_sum(const float *__restrict__ part, int i) {
    float s = 0.f;
#pragma unroll
    for (int sl = 0; sl < MLP_SLICES; ++sl) s += part[sl * MLP_P + i];
    return s;
}

__global__ void k_mlp_grad(const float *__restrict__ part, float *__restrict__ g) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < MLP_P) g[i] = mlp_grad_sum(part, i);
}

// Adam on the gradient summed from the slices.
__global__ void k_mlp_adam(float *__restrict__ theta, const float *__restrict__ part, float *__restrict__ m,
                           float *__restrict__ v, _Float16 *__restrict__ w16, float lr, float b1, float b2,
                           float eps, float bc1, float bc2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= MLP_P) return;
    const float gi = mlp_grad_sum(part, i);
    const float mi = fmaf(1.f - b1, gi, b1 * m[i]);
    const float vi = fmaf(gi, (1.f - b2) * gi, b2 * v[i]);
    m[i] = mi;
    v[i] = vi;
    const float th = theta[i] - lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
    theta[i] = th;
    w16[i] = (_Float16)th;
}

// features and target (q, 0, 0, 0) of each link of the list
__global__ void k_mlp_collect(Params p, const DevParticle *__restrict__ P, const float *__restrict__ body,
                              const uint32_t *__restrict__ l_node, const uint32_t *__restrict__ l_do,
                              const double *__restrict__ l_q, int n, _Float16 *__restrict__ feat,
                              float *__restrict__ target) {
    const int l = blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= n) return;
    const long long node = l_node[l];
    const int i = (int)(l_do[l] & 31u), pid = (int)(l_do[l] >> 8);
    _Float16 *f = feat + (long long)l * MLP_IN;
    float *t = target + (long long)l * MLP_OUT;
    if (node >= p.N || pid >= p.np || i < 1 || i >= 19) {  // never expected: an all-zero sample
        for (int a = 0; a < MLP_IN; ++a) f[a] = (_Float16)0.f;
        for (int a = 0; a < MLP_OUT; ++a) t[a] = 0.f;
        return;
    }
    const int x = (int)(node % p.nx), y = (int)((node / p.nx) % p.ny), z = (int)(node / ((long long)p.nx * p.ny));
    const int e[3] = {m_ex[i], m_ey[i], m_ez[i]};
    double head[7];
    mlp_link_head(p, P[pid], x, y, z, e, head);
    for (int a = 0; a < 7; ++a) f[a] = (_Float16)head[a];
    for (int c = 0; c < MLP_BODY; ++c) f[7 + c] = (_Float16)body[pid * MLP_BODY + c];
    t[0] = (float)l_q[l];
    t[1] = t[2] = t[3] = 0.f;
}

// Closest-point samples, one block scanning the pair slots in order: a
// converged pair (i < j) gets the next sample (block prefix of the flags),
// inputs from body i with the partner's centroid as the query point, target
// outputs 1..3 = the stationary point in body i's frame scaled by
// 1/sqrt(sum k) (output 0 untargeted).
__global__ __launch_bounds__(1024) void k_mlp_collect_contact(Params p, const DevParticle *__restrict__ P,
                                                              const float *__restrict__ body, ContactBufs cb,
                                                              int n_max, _Float16 *__restrict__ feat,
                                                              float *__restrict__ target, Counters *cnt) {
    __shared__ int wsum[16];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int np = p.np;
    const long long np2 = (long long)np * np;
    int base = 0;
    for (long long q0 = 0; q0 < np2; q0 += 1024) {
        const long long q = q0 + t;
        int i = 0, j = 0;
        bool ok = false;
        if (q < np2) {
            i = (int)(q / np);
            j = (int)(q - (long long)i * np);
            ok = j > i && cb.pairOk[q];
        }
        int incl = ok ? 1 : 0;
        for (int d = 1; d < 64; d <<= 1) {
            const int v = __shfl_up(incl, d);
            if (lane >= d) incl += v;
        }
        if (lane == 63) wsum[wv] = incl;
        __syncthreads();
        int wb = 0, tot = 0;
        for (int k = 0; k < 16; ++k) {
            if (k < wv) wb += wsum[k];
            tot += wsum[k];
        }
        const int idx = base + wb + incl - (ok ? 1 : 0);
        if (ok && idx < n_max) {
            _Float16 *f = feat + (long long)idx * MLP_IN;
            float *tg = target + (long long)idx * MLP_OUT;
            double head[7];
            mlp_contact_head(p, P[i], P[j], head);
            for (int a = 0; a < 7; ++a) f[a] = (_Float16)head[a];
            for (int c = 0; c < MLP_BODY; ++c) f[7 + c] = (_Float16)body[i * MLP_BODY + c];
            const int zero[3] = {0, 0, 0};
            double off[7];
            mlp_point_head(p, P[i], cb.pairXm + 3 * q, zero, 1.0, off);
            tg[0] = 0.f;
            for (int a = 0; a < 3; ++a) tg[1 + a] = (float)off[a];
        }
        base += tot;
        __syncthreads();  // wsum is written again
    }
    if (t == 0) cnt->n_collect = min(base, n_max);
}

static int cdiv(long long a, long long b) { return (int)((a + b - 1) / b); }

void launch_mlp_init(const MlpBlob &b, hipStream_t s) {
    k_mlp_init<<<cdiv(MLP_P, 256), 256, 0, s>>>(b.theta, b.m, b.v, b.w16, b.t);
}

template <typename TA, typename TW>
static void forward_t(const MlpBlob &b, const TA *X, const TW *W, int n, hipStream_t s) {
    TA *h1 = (TA *)b.h1, *h2 = (TA *)b.h2;
    k_mlp_layer<TA, TW><<<cdiv((long long)n * MLP_H, 256), 256, 0, s>>>(X, MLP_IN, W, MLP_OFF_W1, MLP_OFF_B1, MLP_H,
                                                                        n, h1, nullptr);
    k_mlp_layer<TA, TW><<<cdiv((long long)n * MLP_H, 256), 256, 0, s>>>(h1, MLP_H, W, MLP_OFF_W2, MLP_OFF_B2, MLP_H,
                                                                        n, h2, nullptr);
    k_mlp_layer<TA, TW><<<cdiv((long long)n * MLP_OUT, 256), 256, 0, s>>>(h2, MLP_H, W, MLP_OFF_W3, MLP_OFF_B3,
                                                                          MLP_OUT, n, nullptr, b.out);
}

// Forward pass of 32 samples per block with the matrix-core hidden layers
// (the link solver's form): outputs [n][4] into out.
// Wave inference: each wave loads the network once and takes tiles of 32
// samples (grid stride).
__global__ __launch_bounds__(256) void k_mlp_forward_mfma(const _Float16 *__restrict__ X,
                                                          const _Float16 *__restrict__ w, int n,
                                                          float *__restrict__ out) {
    const int lane = threadIdx.x & 63, s = lane & 31, h = lane >> 5;
    const int wv = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6), nw = gridDim.x * (blockDim.x >> 6);
    if (wv * 32 >= n) return;  // wave-uniform; no block barrier in this kernel
    MlpWave W;
    mlp_wave_load(W, w);
    _Float16 w3[MLP_OUT][32];
    float b3[MLP_OUT];
#pragma unroll
    for (int o = 0; o < MLP_OUT; ++o) {
        mlp_wave_load_out(w3[o], w, o);
        b3[o] = (float)w[MLP_OFF_B3 + o];
    }
    for (int r0 = wv * 32; r0 < n; r0 += nw * 32) {
        const int r = r0 + s;
        const bool ok = r < n;
        const _Float16 *xr = X + (long long)(ok ? r : 0) * MLP_IN;
        mlp_h8 x[MLP_S1];
#pragma unroll
        for (int m = 0; m < MLP_S1; ++m)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = mlp_l1_input(2 * m + h, e);
                const _Float16 v = xr[k >= 0 ? k : 0];
                x[m][e] = k >= 0 ? (ok ? v : (_Float16)0.f) : (k == -1 ? (_Float16)1.f : (_Float16)0.f);
            }
        float z[MLP_OUT];
        mlp_wave_forward<MLP_OUT>(W, x, w3, b3, z);
#pragma unroll
        for (int o = 0; o < MLP_OUT; ++o)
            if (ok && h == (o & 1)) out[(long long)r * MLP_OUT + o] = z[o];
    }
}

void launch_mlp_forward(const MlpBlob &b, const void *X, int n, int precision, hipStream_t s) {
    if (precision == 1) forward_t<float, float>(b, (const float *)X, b.theta, n, s);
    else if (precision == 2) {
        if (n > 0) k_mlp_forward_mfma<<<min(cdiv(n, 128), 1024), 256, 0, s>>>((const _Float16 *)X, b.w16, n, b.out);
    } else forward_t<_Float16, _Float16>(b, (const _Float16 *)X, b.w16, n, s);
}

// The batch's gradient in slices (b.h1 holds them: 16 P of its 262 144 values).
static_assert(MLP_SLICES * MLP_P <= MLP_MAX_BATCH * MLP_H, "the slices fit the activation workspace");
static void slices(const MlpBlob &b, const void *X, const float *T, int n, int precision, float *sq, hipStream_t s) {
    auto run = [&](auto kernel, auto x, auto w) { kernel<<<MLP_SLICES, MLP_BLK, 0, s>>>(x, w, T, n, b.h1, sq); };
    const bool full = n % (MLP_SLICES * MLP_T) == 0;
    if (precision == 1)
        run(full ? k_mlp_slice<float, float, true> : k_mlp_slice<float, float, false>, (const float *)X, b.theta);
    else
        run(full ? k_mlp_slice<_Float16, _Float16, true> : k_mlp_slice<_Float16, _Float16, false>, (const _Float16 *)X,
            b.w16);
}

void launch_mlp_loss_grad(const MlpBlob &b, const void *X, const float *T, int n, int precision, hipStream_t s) {
    slices(b, X, T, n, precision, b.sq, s);
    k_mlp_loss<<<1, 256, 0, s>>>(b.sq, n * MLP_OUT, n, b.loss);
    k_mlp_grad<<<cdiv(MLP_P, 256), 256, 0, s>>>(b.h1, b.g);
}

void launch_mlp_adam_step(const MlpBlob &b, const void *X, const float *T, int n, int precision, float lr, float beta1,
                          float beta2, float eps, float bc1, float bc2, hipStream_t s) {
    slices(b, X, T, n, precision, nullptr, s);
    k_mlp_adam<<<cdiv(MLP_P, 64), 64, 0, s>>>(b.theta, b.h1, b.m, b.v, b.w16, lr, beta1, beta2, eps, bc1, bc2);
}

void launch_mlp_collect_contact(const Params &p, const DevParticle *P, const float *body, const ContactBufs &cb,
                                int n_max, _Float16 *feat, float *target, Counters *cnt, hipStream_t s) {
    k_mlp_collect_contact<<<1, 1024, 0, s>>>(p, P, body, cb, n_max, feat, target, cnt);
}

void launch_mlp_collect(const Params &p, const DevParticle *P, const float *body, const uint32_t *l_node,
                        const uint32_t *l_do, const double *l_q, int n, _Float16 *feat, float *target,
                        hipStream_t s) {
    if (n > 0) k_mlp_collect<<<cdiv(n, 256), 256, 0, s>>>(p, P, body, l_node, l_do, l_q, n, feat, target);
}

}  // namespace mdl
