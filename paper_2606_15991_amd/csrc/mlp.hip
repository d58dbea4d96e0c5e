// mlp.hip -- training kernels of the tile-picker cost model: a multilayer
// perceptron with `depth` hidden ReLU layers of `hidden` units and one linear
// output, regressing log(time) of a (shape, configuration) pair.
//
// Forward:  H_0 = X,  H_l = relu(H_{l-1} W_l^T + b_l),  out = H_depth w^T + b
// Loss:     L = (1/B) sum_b (out_b - y_b)^2
// Backward: dZ_out = 2 (out - y) / B; for each layer, dW = dZ^T H_prev,
//           db = column sums of dZ, dH_prev = dZ W masked by H_prev > 0.
// Every reduction runs in a fixed order in one thread or one workgroup:
// no atomics, identical results on every run.  Parameters per layer are W
// (out x in, row-major) followed by b (out).
#include <math.h>

#include <algorithm>

#include "host_internal.hpp"
#include "tg_device.hpp"

namespace tg {
namespace {

// Y[b][o] = act(sum_i X[b][i] W[o][i] + bias[o])
__global__ void dense_fwd(const float *__restrict__ X,
                          const float *__restrict__ W,
                          const float *__restrict__ bias, float *__restrict__ Y,
                          int batch, int in, int out, int relu) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)batch * out) return;
    const int b = (int)(e / out), o = (int)(e % out);
    float s = bias[o];
    const float *x = X + (int64_t)b * in;
    const float *w = W + (int64_t)o * in;
    for (int i = 0; i < in; ++i) s = fmaf(x[i], w[i], s);
    Y[e] = (relu && s < 0.f) ? 0.f : s;
}

// dZ[b] = 2 (out[b] - y[b]) / B and loss = (1/B) sum (out - y)^2, one
// workgroup, fixed order.
__global__ __launch_bounds__(256) void loss_grad(const float *__restrict__ out,
                                                 const float *__restrict__ y,
                                                 float *__restrict__ dz,
                                                 float *__restrict__ loss,
                                                 int batch) {
    __shared__ float part[256];
    float s = 0.f;
    const float inv = 1.0f / (float)batch;
    for (int b = threadIdx.x; b < batch; b += 256) {
        const float d = out[b] - y[b];
        dz[b] = 2.0f * d * inv;
        s = fmaf(d, d, s);
    }
    part[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = part[0] * inv;
}

// dW[o][i] = sum_b dZ[b][o] H[b][i]  (i < in);  db[o] = sum_b dZ[b][o]
// (thread i == in).  One thread per output entry, batch summed in order.
__global__ void dense_bwd_weight(const float *__restrict__ dZ,
                                 const float *__restrict__ H,
                                 float *__restrict__ dW,
                                 float *__restrict__ db, int batch, int in,
                                 int out) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= out * (in + 1)) return;
    const int o = e / (in + 1), i = e % (in + 1);
    float s = 0.f;
    if (i < in) {
        for (int b = 0; b < batch; ++b)
            s = fmaf(dZ[(int64_t)b * out + o], H[(int64_t)b * in + i], s);
        dW[(int64_t)o * in + i] = s;
    } else {
        for (int b = 0; b < batch; ++b) s += dZ[(int64_t)b * out + o];
        db[o] = s;
    }
}

// dH[b][i] = (H[b][i] > 0) * sum_o dZ[b][o] W[o][i]
__global__ void dense_bwd_input(const float *__restrict__ dZ,
                                const float *__restrict__ W,
                                const float *__restrict__ H,
                                float *__restrict__ dH, int batch, int in,
                                int out) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)batch * in) return;
    const int b = (int)(e / in), i = (int)(e % in);
    if (!(H[e] > 0.f)) {
        dH[e] = 0.f;
        return;
    }
    float s = 0.f;
    for (int o = 0; o < out; ++o)
        s = fmaf(dZ[(int64_t)b * out + o], W[(int64_t)o * in + i], s);
    dH[e] = s;
}

// Adam (Kingma & Ba): m = b1 m + (1-b1) g; v = b2 v + (1-b2) g^2;
// p -= lr * (m / (1 - b1^t)) / (sqrt(v / (1 - b2^t)) + eps)
// The constants 1 - b1, 1 - b2 and the bias corrections are formed in
// binary64 on the host: 1 - 0.999 in binary32 loses 4 significant digits.
__global__ void adam_step(float *__restrict__ p, const float *__restrict__ g,
                          float *__restrict__ m, float *__restrict__ v,
                          int64_t n, float lr, float b1, float b2, float omb1,
                          float omb2, float eps, float c1, float c2) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const float gi = g[e];
    const float mi = b1 * m[e] + omb1 * gi;
    const float vi = b2 * v[e] + omb2 * (gi * gi);
    m[e] = mi;
    v[e] = vi;
    p[e] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// ------------------------------------------------------ fused small network
//
// Networks of at most 64 inputs and 64 hidden units (the picker's own is 24
// inputs, 3 x 64 hidden): forward, loss and backward of a 32-row batch tile
// in one workgroup.  Weights, activations and their gradients stay in LDS;
// the weight gradients accumulate in matrix-core registers over all tiles
// of the workgroup, which stores one partial gradient at the end; a second
// launch sums the partials in workgroup order.  All arithmetic is binary32
// (v_mfma_f32_16x16x4_f32) and in a fixed order: no atomics.
//
// Bound: 1.1 GFLOP of binary32 products at a batch of 20000, and about ten
// dependent LDS round trips per tile; one workgroup of eight wavefronts per
// compute unit (the weights are read from global memory once per compute
// unit).  Measured at 20000 x 24, 3 x 64 hidden, with Adam: 33.6 ms a step
// layer by layer (the weight gradients alone 33.1 ms: one thread walked the
// whole batch per entry), 40 us fused.
//
// LDS rows are 68 floats, so that neither 16-byte reads along a row nor dword
// reads down a column fall on few banks; 19 % of the LDS cycles are conflicts
// all the same.  Wavefronts wait 56 % of their time and the matrix cores are
// busy 29 % (counters at 20000 x 24, 3 x 64).
constexpr int kMlpW = 64;            // padded layer width
constexpr int kMlpLd = 68;           // LDS row stride
constexpr int kMlpRows = 32;         // batch rows per tile
constexpr int kMlpThreads = 512;
constexpr int kMlpMaxDepth = 4;      // LDS and accumulator registers

struct MlpArgs {
    const float *params, *X, *y;
    float *out;       // forward: batch values
    float *part;      // backward: gridDim.x partial gradients of n_par + 1
    float *grads;     // backward, one workgroup: the gradient itself
    float *loss;
    int n_in, hidden, batch, tiles, n_par;
};

constexpr int mlp_smem(int depth) {
    return 4 * (depth * kMlpW * kMlpLd + depth * kMlpW + kMlpW + 4 +
                (depth + 1) * kMlpRows * kMlpLd + kMlpRows + kMlpThreads);
}

__device__ __forceinline__ f32x4 mfma16_f32(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 lds4(const float *p) {
    return *reinterpret_cast<const f32x4 *>(p);
}

template <int DEPTH, bool BWD>
__global__ __launch_bounds__(kMlpThreads) void mlp_fused(MlpArgs g) {
    extern __shared__ __align__(16) float sm[];
    constexpr int WL = kMlpW * kMlpLd, AL = kMlpRows * kMlpLd;
    float *W = sm;                                  // [DEPTH][64][68]
    float *bias = W + DEPTH * WL;                   // [DEPTH][64]
    float *wout = bias + DEPTH * kMlpW;             // [64], then the bias
    float *act = wout + kMlpW + 4;                  // [DEPTH + 1][32][68]
    float *dz = act + (DEPTH + 1) * AL;             // [32]
    float *red = dz + kMlpRows;                     // [512]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lr = lane & 15, q4 = lane >> 4;
    const int H = g.hidden;
    {
        const float *p = g.params;
#pragma unroll
        for (int l = 0; l < DEPTH; ++l) {
            const int in = l == 0 ? g.n_in : H;
            for (int e = tid; e < kMlpW * kMlpW; e += kMlpThreads) {
                const int o = e >> 6, i = e & 63;
                W[l * WL + o * kMlpLd + i] =
                    o < H && i < in ? p[o * in + i] : 0.f;
            }
            if (tid < kMlpW)
                bias[l * kMlpW + tid] = tid < H ? p[H * in + tid] : 0.f;
            p += H * in + H;
        }
        if (tid < kMlpW) wout[tid] = tid < H ? p[tid] : 0.f;
        if (tid == kMlpW) wout[kMlpW] = p[H];
    }
    const float inv = 1.0f / (float)g.batch;
    const int kc0 = (g.n_in + 15) >> 4, kch = (H + 15) >> 4;
    // fixed roles: forward / input gradients, one 16 x 16 tile per wavefront
    const int mt = (wave >> 2) * 16, nt = (wave & 3) * 16;
    const bool pad = nt + lr >= H;
    // weight gradients, two 16 x 16 tiles per wavefront and layer
    const int ot = (wave >> 1) * 16, it = (wave & 1) * 32;
    // column sums: column tid % 64 over the four rows of part tid / 64
    const int ci = tid & 63, cr = (tid >> 6) * 4;
    f32x4 dw[DEPTH][2];
    float db[DEPTH], dwo = 0.f, dbo = 0.f, ls = 0.f;
#pragma unroll
    for (int l = 0; l < DEPTH; ++l) {
        dw[l][0] = dw[l][1] = f32x4{0.f, 0.f, 0.f, 0.f};
        db[l] = 0.f;
    }
    for (int t = blockIdx.x; t < g.tiles; t += gridDim.x) {
        const int r0 = t * kMlpRows;
        const int valid = min(kMlpRows, g.batch - r0);
#pragma unroll
        for (int u = 0; u < kMlpRows * kMlpW / kMlpThreads; ++u) {
            const int e = u * kMlpThreads + tid, r = e >> 6, i = e & 63;
            act[r * kMlpLd + i] =
                r < valid && i < g.n_in ? g.X[(int64_t)(r0 + r) * g.n_in + i]
                                        : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int l = 0; l < DEPTH; ++l) {
            const float *A = act + l * AL + (mt + lr) * kMlpLd + 4 * q4;
            const float *B = W + l * WL + (nt + lr) * kMlpLd + 4 * q4;
            const float b0 = bias[l * kMlpW + nt + lr];
            f32x4 acc = {b0, b0, b0, b0};
            const int kc = l == 0 ? kc0 : kch;
            for (int j = 0; j < kc; ++j) {
                const f32x4 a = lds4(A + 16 * j), b = lds4(B + 16 * j);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc = mfma16_f32(a[e], b[e], acc);
            }
            float *Y = act + (l + 1) * AL + nt + lr;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = mt + 4 * q4 + v;
                const float s = acc[v];
                // rows past the batch and columns past the layer stay zero
                // (zero weights alone would make them NaN behind an infinity)
                Y[r * kMlpLd] = r >= valid || pad || s < 0.f ? 0.f : s;
            }
            __syncthreads();
        }
        float *HL = act + DEPTH * AL;
        {
            const int r = tid >> 4, q = tid & 15;
            const f32x4 h = lds4(HL + r * kMlpLd + 4 * q);
            const f32x4 w = lds4(wout + 4 * q);
            float s = h[0] * w[0];
#pragma unroll
            for (int e = 1; e < 4; ++e) s = fmaf(h[e], w[e], s);
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) s += __shfl_xor(s, o);
            if (q == 0) {
                s += wout[kMlpW];
                if constexpr (BWD) {
                    const float d = r < valid ? s - g.y[r0 + r] : 0.f;
                    dz[r] = 2.0f * d * inv;
                    ls = fmaf(d, d, ls);
                } else if (r < valid) {
                    g.out[r0 + r] = s;
                }
            }
        }
        __syncthreads();
        if constexpr (BWD) {
            // output layer: its gradients, and dZ of the last hidden layer
            // in place of its activations
            if (tid < kMlpRows) dbo += dz[tid];
            const float w = wout[ci];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                float *hp = HL + (cr + k) * kMlpLd + ci;
                const float h = *hp, d = dz[cr + k];
                dwo = fmaf(d, h, dwo);
                *hp = h > 0.f ? d * w : 0.f;
            }
            __syncthreads();
#pragma unroll
            for (int l = DEPTH - 1; l >= 0; --l) {
                const float *dZ = act + (l + 1) * AL;
                float *Hp = act + l * AL;
#pragma unroll
                for (int k = 0; k < 4; ++k) db[l] += dZ[(cr + k) * kMlpLd + ci];
#pragma unroll
                for (int j = 0; j < kMlpRows / 16; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int k = (16 * j + 4 * q4 + e) * kMlpLd;
                        const float a = dZ[k + ot + lr];
                        dw[l][0] = mfma16_f32(a, Hp[k + it + lr], dw[l][0]);
                        dw[l][1] = mfma16_f32(a, Hp[k + it + 16 + lr],
                                              dw[l][1]);
                    }
                if (l > 0) {
                    const float *A = dZ + (mt + lr) * kMlpLd + 4 * q4;
                    const float *B = W + l * WL + nt + lr;
                    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
                    for (int j = 0; j < kch; ++j) {
                        const f32x4 a = lds4(A + 16 * j);
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            acc = mfma16_f32(
                                a[e], B[(16 * j + 4 * q4 + e) * kMlpLd], acc);
                    }
                    __syncthreads();   // Hp has been read by every wavefront
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        float *hp = Hp + (mt + 4 * q4 + v) * kMlpLd + nt + lr;
                        *hp = *hp > 0.f ? acc[v] : 0.f;
                    }
                }
                __syncthreads();
            }
        }
    }
    if constexpr (BWD) {
        const bool direct = gridDim.x == 1;
        float *dst = direct ? g.grads
                            : g.part + (int64_t)blockIdx.x * (g.n_par + 1);
        // column sums of the eight row parts, in part order
        auto fold = [&](float v, float *to) {
            red[tid] = v;
            __syncthreads();
            if (tid < H) {
                float s = red[tid];
#pragma unroll
                for (int p = 1; p < kMlpThreads / kMlpW; ++p)
                    s += red[p * kMlpW + tid];
                to[tid] = s;
            }
            __syncthreads();
        };
#pragma unroll
        for (int l = 0; l < DEPTH; ++l) {
            const int in = l == 0 ? g.n_in : H;
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int o = ot + 4 * q4 + v, i = it + 16 * c + lr;
                    if (o < H && i < in) dst[o * in + i] = dw[l][c][v];
                }
            fold(db[l], dst + H * in);
            dst += H * in + H;
        }
        fold(dwo, dst);
        red[tid] = ls;                       // lanes tid % 16 == 0
        if (tid < kMlpRows) dz[tid] = dbo;
        __syncthreads();
        if (tid == 0) {
            float s = 0.f, b = 0.f;
            for (int r = 0; r < kMlpRows; ++r) {
                s += red[16 * r];
                b += dz[r];
            }
            dst[H] = b;
            if (direct)
                *g.loss = s * inv;
            else
                dst[H + 1] = s;
        }
    }
}

// grads[p] = sum over the partials in workgroup order (four interleaved
// quarters per workgroup of 64 entries, folded in order); the entry after
// the last parameter is the loss sum.
__global__ __launch_bounds__(256) void mlp_fold(const float *__restrict__ part,
                                                int n_part, int n_par,
                                                float *__restrict__ grads,
                                                float *__restrict__ loss,
                                                float inv) {
    __shared__ float red[4][64];
    const int c = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int p = blockIdx.x * 64 + c;
    const int64_t ld = n_par + 1;
    const int per = (n_part + 3) / 4;
    const int b0 = q * per, b1 = min(n_part, b0 + per);
    float s = 0.f;
    if (p <= n_par) {
        const float *src = part + p;
        int b = b0;
        for (; b + 8 <= b1; b += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = src[(b + u) * ld];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; b < b1; ++b) s += src[b * ld];
    }
    red[q][c] = s;
    __syncthreads();
    if (q == 0 && p <= n_par) {
        s = ((red[0][c] + red[1][c]) + red[2][c]) + red[3][c];
        if (p < n_par)
            grads[p] = s;
        else
            *loss = s * inv;
    }
}

inline unsigned blocks_for(int64_t n, int t) {
    return (unsigned)((n + t - 1) / t);
}

struct Layout {
    int n_in, hidden, depth, batch;
    // parameter offsets of layer l's W and b (l = 0 .. depth; depth = output)
    size_t w_off(int l) const {
        size_t off = 0;
        int in = n_in;
        for (int k = 0; k < l; ++k) {
            const int out = k < depth ? hidden : 1;
            off += (size_t)out * in + out;
            in = out;
        }
        return off;
    }
    int in_of(int l) const { return l == 0 ? n_in : hidden; }
    int out_of(int l) const { return l < depth ? hidden : 1; }
    // workspace: H_1..H_depth (batch x hidden each), out (batch), two dZ
    // buffers (batch x hidden), the loss
    size_t ws_floats() const {
        return (size_t)depth * batch * hidden + batch +
               2 * (size_t)batch * hidden + 4;
    }
};

hipError_t forward(const Layout &L, const float *params, const float *X,
                   float *ws, float *out, hipStream_t st) {
    const float *prev = X;
    for (int l = 0; l <= L.depth; ++l) {
        const int in = L.in_of(l), o = L.out_of(l);
        const float *W = params + L.w_off(l);
        const float *b = W + (size_t)o * in;
        float *Y = l < L.depth ? ws + (size_t)l * L.batch * L.hidden : out;
        hipLaunchKernelGGL(dense_fwd, dim3(blocks_for((int64_t)L.batch * o,
                                                      256)),
                           dim3(256), 0, st, prev, W, b, Y, L.batch, in, o,
                           l < L.depth ? 1 : 0);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        prev = Y;
    }
    return hipSuccess;
}

// The fused kernels take networks whose layers fit 64 columns and whose
// weights and activations fit LDS (kMlpMaxDepth); wider or deeper ones run
// layer by layer.
bool fused_ok(const Layout &L) {
    return L.n_in <= kMlpW && L.hidden <= kMlpW && L.depth <= kMlpMaxDepth;
}

template <int DEPTH, bool BWD>
hipError_t launch_fused_depth(const MlpArgs &a, int grid, hipStream_t st) {
    const void *k = reinterpret_cast<const void *>(&mlp_fused<DEPTH, BWD>);
    // LDS beyond the 64 KiB default
    hipError_t e = hipFuncSetAttribute(
        k, hipFuncAttributeMaxDynamicSharedMemorySize, mlp_smem(DEPTH));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((mlp_fused<DEPTH, BWD>), dim3(grid), dim3(kMlpThreads),
                       mlp_smem(DEPTH), st, a);
    return hipGetLastError();
}

template <bool BWD>
hipError_t launch_fused(const Layout &L, const MlpArgs &a, int grid,
                        hipStream_t st) {
    static_assert(mlp_smem(kMlpMaxDepth) <= 163840, "160 KiB of LDS");
    switch (L.depth) {
    case 1: return launch_fused_depth<1, BWD>(a, grid, st);
    case 2: return launch_fused_depth<2, BWD>(a, grid, st);
    case 3: return launch_fused_depth<3, BWD>(a, grid, st);
    case 4: return launch_fused_depth<4, BWD>(a, grid, st);
    default: return hipErrorInvalidValue;
    }
}

MlpArgs fused_args(const Layout &L, const float *params, const float *X) {
    MlpArgs a{};
    a.params = params;
    a.X = X;
    a.n_in = L.n_in;
    a.hidden = L.hidden;
    a.batch = L.batch;
    a.tiles = (int)(((int64_t)L.batch + kMlpRows - 1) / kMlpRows);
    a.n_par = (int)L.w_off(L.depth + 1);
    return a;
}

// One workgroup per compute unit (LDS holds one).
int fused_grid(const MlpArgs &a) {
    const int cus = tg_device_cus();
    return std::min(a.tiles, cus > 0 ? cus : 256);
}

}  // namespace
}  // namespace tg

using namespace tg;

extern "C" {

size_t tile_mlp_workspace_bytes(int32_t n_in, int32_t hidden, int32_t depth,
                                int32_t batch) {
    if (n_in <= 0 || hidden <= 0 || depth <= 0 || batch <= 0) return 0;
    Layout L{n_in, hidden, depth, batch};
    return L.ws_floats() * sizeof(float);
}

static tg_status check_mlp(const float *params, int32_t n_in, int32_t hidden,
                           int32_t depth, const float *X, int32_t batch,
                           void *ws, size_t ws_bytes) {
    if (!params || !X || n_in <= 0 || hidden <= 0 || depth <= 0 || batch <= 0)
        return TG_E_ARG;
    if (!ws || ws_bytes < tile_mlp_workspace_bytes(n_in, hidden, depth, batch))
        return TG_E_WORKSPACE;
    return TG_OK;
}

tg_status tile_mlp_forward(const float *params, int32_t n_in, int32_t hidden,
                           int32_t depth, const float *X, int32_t batch,
                           float *out, void *ws, size_t ws_bytes,
                           tg_stream stream) {
    tg_status st = check_mlp(params, n_in, hidden, depth, X, batch, ws,
                             ws_bytes);
    if (st != TG_OK) return st;
    if (!out) return TG_E_ARG;
    Layout L{n_in, hidden, depth, batch};
    hipStream_t hs = static_cast<hipStream_t>(stream);
    if (fused_ok(L)) {
        MlpArgs a = fused_args(L, params, X);
        a.out = out;
        return launch_fused<false>(L, a, fused_grid(a), hs) == hipSuccess
                   ? TG_OK : TG_E_HIP;
    }
    hipError_t e = forward(L, params, X, static_cast<float *>(ws), out, hs);
    return e == hipSuccess ? TG_OK : TG_E_HIP;
}

tg_status tile_mlp_loss_grad(const float *params, int32_t n_in,
                             int32_t hidden, int32_t depth, const float *X,
                             const float *y, int32_t batch, float *grads,
                             float *loss, void *ws, size_t ws_bytes,
                             tg_stream stream) {
    tg_status st = check_mlp(params, n_in, hidden, depth, X, batch, ws,
                             ws_bytes);
    if (st != TG_OK) return st;
    if (!y || !grads || !loss) return TG_E_ARG;
    hipStream_t hs = static_cast<hipStream_t>(stream);
    Layout L{n_in, hidden, depth, batch};
    float *w = static_cast<float *>(ws);
    if (fused_ok(L)) {
        MlpArgs a = fused_args(L, params, X);
        a.y = y;
        a.part = w;
        a.grads = grads;
        a.loss = loss;
        // as many partial gradients as the workspace holds; where it holds
        // fewer than two (batches below about 64), one workgroup stores the
        // gradient itself
        const size_t fit = L.ws_floats() / ((size_t)a.n_par + 1);
        const int grid = (int)std::max<size_t>(
            1, std::min<size_t>(fit, (size_t)fused_grid(a)));
        hipError_t e = launch_fused<true>(L, a, grid, hs);
        if (e == hipSuccess && grid > 1) {
            hipLaunchKernelGGL(mlp_fold, dim3(blocks_for(a.n_par + 1, 64)),
                               dim3(256), 0, hs, w, grid, a.n_par, grads,
                               loss, 1.0f / (float)batch);
            e = hipGetLastError();
        }
        return e == hipSuccess ? TG_OK : TG_E_HIP;
    }
    float *acts = w;                                        // H_1..H_depth
    float *out = w + (size_t)depth * batch * hidden;        // batch
    float *dz0 = out + batch;                               // batch x hidden
    float *dz1 = dz0 + (size_t)batch * hidden;              // batch x hidden
    hipError_t e = forward(L, params, X, w, out, hs);
    if (e != hipSuccess) return TG_E_HIP;
    hipLaunchKernelGGL(loss_grad, dim3(1), dim3(256), 0, hs, out, y, dz0, loss,
                       batch);
    if ((e = hipGetLastError()) != hipSuccess) return TG_E_HIP;
    float *dz = dz0, *dprev = dz1;
    for (int l = depth; l >= 0; --l) {
        const int in = L.in_of(l), o = L.out_of(l);
        const float *H = l == 0 ? X : acts + (size_t)(l - 1) * batch * hidden;
        const float *W = params + L.w_off(l);
        float *dW = grads + L.w_off(l);
        float *db = dW + (size_t)o * in;
        hipLaunchKernelGGL(dense_bwd_weight, dim3(blocks_for(o * (in + 1), 256)),
                           dim3(256), 0, hs, dz, H, dW, db, batch, in, o);
        if ((e = hipGetLastError()) != hipSuccess) return TG_E_HIP;
        if (l > 0) {
            hipLaunchKernelGGL(dense_bwd_input,
                               dim3(blocks_for((int64_t)batch * in, 256)),
                               dim3(256), 0, hs, dz, W, H, dprev, batch, in, o);
            if ((e = hipGetLastError()) != hipSuccess) return TG_E_HIP;
            float *t = dz;
            dz = dprev;
            dprev = t;
        }
    }
    return TG_OK;
}

tg_status tile_mlp_adam(float *params, const float *grads, float *m, float *v,
                        int64_t n, double lr, double beta1, double beta2,
                        double eps, int32_t t, tg_stream stream) {
    if (!params || !grads || !m || !v || n < 0 || t < 1) return TG_E_ARG;
    if (n == 0) return TG_OK;
    const float c1 = (float)(1.0 - pow(beta1, (double)t));
    const float c2 = (float)(1.0 - pow(beta2, (double)t));
    hipLaunchKernelGGL(adam_step, dim3(blocks_for(n, 256)), dim3(256), 0,
                       static_cast<hipStream_t>(stream), params, grads, m, v,
                       n, (float)lr, (float)beta1, (float)beta2,
                       (float)(1.0 - beta1), (float)(1.0 - beta2), (float)eps,
                       c1, c2);
    return hipGetLastError() == hipSuccess ? TG_OK : TG_E_HIP;
}

}  // extern "C"
