// split_norm.hip -- two memory-bound helpers of the product path.
//
// (1) Split of binary32 operands into bfloat16 planes for the BF16x3 / BF16x6
//     precisions:  hi = bf16(a), mid = bf16(a - hi), lo = bf16(a - hi - mid),
//     each rounded to nearest even (the residuals are exact in binary32).
//     Plane block b of the destination receives plane order[b], so a single
//     bf16 product over the concatenated K axis sums the chosen plane
//     products into one binary32 accumulator.
// (2) Binary64 reductions of the relative Frobenius error of a result
//     against a binary64 reference (the only binary64 arithmetic on the GPU):
//     fixed-order two-pass reduction, no atomics, deterministic.
#include "tg_device.hpp"
#include "tg_internal.hpp"

namespace tg {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Planes of V consecutive elements (V = 8: 16-byte accesses, needs rows,
// row strides and plane strides of whole chunks).  Bound by memory: 4 bytes
// read and 2 per plane block written for each element; one element a lane
// and a copy of a plane for every product ran two operands of 4096 x 4096
// into six blocks in 150 us; three planes each, stored once, take 52.
template <int V>
__device__ __forceinline__ void split_chunks(const SplitArgs &s,
                                             int64_t first, int64_t step) {
    const uint32_t per_row = (uint32_t)(s.cols / V);
    const int64_t total = (int64_t)s.rows * per_row;
    for (int64_t e = first; e < total; e += step) {
        int64_t i, j;
        if (total <= UINT32_MAX) {
            i = (uint32_t)e / per_row;
            j = ((uint32_t)e - (uint32_t)i * per_row) * (int64_t)V;
        } else {
            i = e / per_row;
            j = (e - i * per_row) * V;
        }
        const float *p = s.src + i * s.ld + j;
        uint16_t *d = s.dst + i * s.ldd + j;
        if constexpr (V == 8) {
            f32x4 x[2] = {*reinterpret_cast<const f32x4 *>(p),
                          *reinterpret_cast<const f32x4 *>(p + 4)};
            u32x4 w[3];
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    const int c = 2 * (h & 1);
                    f32x4 &r = x[h >> 1];
                    const uint32_t v = f32x2_to_bf16x2(r[c], r[c + 1]);
                    w[q][h] = v;
                    r[c] -= bf16_bits_to_f32(v & 0xffffu);
                    r[c + 1] -= bf16_bits_to_f32(v >> 16);
                }
            for (int b = 0; b < s.blocks; ++b) {
                const uint32_t which = (s.order >> (4 * b)) & 0xf;
                *reinterpret_cast<u32x4 *>(d + b * s.plane_stride) =
                    which == 0 ? w[0] : which == 1 ? w[1] : w[2];
            }
        } else {
            const float a = *p;
            uint16_t w[3];
            w[0] = f32_to_bf16_bits(a);
            const float r1 = a - bf16_bits_to_f32(w[0]);
            w[1] = f32_to_bf16_bits(r1);
            const float r2 = r1 - bf16_bits_to_f32(w[1]);
            w[2] = f32_to_bf16_bits(r2);
            for (int b = 0; b < s.blocks; ++b) {
                const uint32_t which = (s.order >> (4 * b)) & 0xf;
                d[b * s.plane_stride] = which == 0   ? w[0]
                                        : which == 1 ? w[1] : w[2];
            }
        }
    }
}

// Both operands in one launch: blocks below na split a, the others b.
template <bool VA, bool VB>
__global__ __launch_bounds__(256) void split_kernel(SplitArgs a, SplitArgs b,
                                                    int na) {
    if ((int)blockIdx.x < na)
        split_chunks<VA ? 8 : 1>(
            a, (int64_t)blockIdx.x * 256 + threadIdx.x, (int64_t)na * 256);
    else
        split_chunks<VB ? 8 : 1>(
            b, (int64_t)(blockIdx.x - na) * 256 + threadIdx.x,
            (int64_t)(gridDim.x - na) * 256);
}

constexpr int NORM_BLOCKS = 256, NORM_THREADS = 256;

__global__ __launch_bounds__(NORM_THREADS) void norm_partial_kernel(
    const void *__restrict__ c, int c_bf16, const double *__restrict__ r,
    int64_t n, double *__restrict__ out) {
    __shared__ double s_num[NORM_THREADS], s_den[NORM_THREADS];
    double num = 0.0, den = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * NORM_THREADS + threadIdx.x; i < n;
         i += (int64_t)NORM_BLOCKS * NORM_THREADS) {
        double cv = c_bf16 ? (double)bf16_bits_to_f32(
                                 static_cast<const uint16_t *>(c)[i])
                           : (double)static_cast<const float *>(c)[i];
        double rv = r[i];
        double d = cv - rv;
        num += d * d;
        den += rv * rv;
    }
    s_num[threadIdx.x] = num;
    s_den[threadIdx.x] = den;
    __syncthreads();
    for (int w = NORM_THREADS / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
            s_num[threadIdx.x] += s_num[threadIdx.x + w];
            s_den[threadIdx.x] += s_den[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[2 + 2 * blockIdx.x] = s_num[0];
        out[3 + 2 * blockIdx.x] = s_den[0];
    }
}

__global__ __launch_bounds__(64) void norm_final_kernel(double *out) {
    if (threadIdx.x != 0) return;
    double num = 0.0, den = 0.0;
    for (int b = 0; b < NORM_BLOCKS; ++b) {
        num += out[2 + 2 * b];
        den += out[3 + 2 * b];
    }
    out[0] = num;
    out[1] = den;
}

}  // namespace

// Whole 16-byte chunks in every row of the source and of every plane.
static bool split_wide(const SplitArgs &s) {
    return s.cols % 8 == 0 && s.ld % 4 == 0 && s.ldd % 8 == 0 &&
           s.plane_stride % 8 == 0 &&
           (reinterpret_cast<uintptr_t>(s.src) |
            reinterpret_cast<uintptr_t>(s.dst)) % 16 == 0;
}

hipError_t launch_split(const SplitArgs &a, const SplitArgs &b,
                        hipStream_t st) {
    const bool va = split_wide(a), vb = split_wide(b);
    const auto blocks = [](const SplitArgs &s, bool wide) {
        const int64_t n = ((int64_t)s.rows * s.cols / (wide ? 8 : 1) + 255) /
                          256;
        return (int)(n < 1 ? 1 : n > 32768 ? 32768 : n);
    };
    const int na = blocks(a, va), nb = blocks(b, vb);
    const auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)(na + nb)), dim3(256), 0,
                           st, a, b, na);
        return hipGetLastError();
    };
    if (va) return vb ? run(split_kernel<true, true>)
                      : run(split_kernel<true, false>);
    return vb ? run(split_kernel<false, true>)
              : run(split_kernel<false, false>);
}

hipError_t launch_error_norm(const void *c, int c_bf16, const double *r,
                             int64_t n, double *out, hipStream_t st) {
    hipLaunchKernelGGL(norm_partial_kernel, dim3(NORM_BLOCKS),
                       dim3(NORM_THREADS), 0, st, c, c_bf16, r, n, out);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(norm_final_kernel, dim3(1), dim3(64), 0, st, out);
    return hipGetLastError();
}

}  // namespace tg
