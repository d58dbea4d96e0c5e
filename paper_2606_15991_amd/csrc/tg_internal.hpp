// tg_internal.hpp -- types shared by the host entry points and the kernels.
//
// The tile schedule below is the single definition of the program ->
// sub-tensor map: the kernels walk it on the device and tile_gemm_plan
// exports it on the host, so the map that tile_partition_check validates is
// the one that runs.  A program is a workgroup, but for the streaming form of
// the decode product: there a workgroup runs several programs in a row
// (skinny_stream says how many), each owning what the map gives it.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <initializer_list>

#include "../../include/tilegemm.h"

namespace tg {

// LDS beyond the 64 KiB default, requested once per kernel and device (an
// attribute of the function on the current device); a request that failed is
// made again by the next launch.
class LdsRequest {
    std::atomic<uint64_t> devices_{0};

public:
    hipError_t operator()(std::initializer_list<const void *> kernels,
                          int bytes) {
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        const uint64_t bit = dev < 64 ? (uint64_t)1 << dev : 0;
        if (devices_.load(std::memory_order_acquire) & bit) return hipSuccess;
        for (const void *k : kernels) {
            if (!k) continue;
            e = hipFuncSetAttribute(
                k, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
            if (e != hipSuccess) return e;
        }
        devices_.fetch_or(bit, std::memory_order_release);
        return hipSuccess;
    }
};

// Programs of one launch are dispatched round-robin over the XCDs of the
// chip (program p lands on XCD p % kXcds).  MI355X has 8.
constexpr int kXcds = 8;

// Output partition and persistent-program count of one launch.
struct Sched {
    int32_t tiles_m, tiles_n;  // ceil(M / bm), ceil(N / bn)
    int32_t n_tiles;           // tiles_m * tiles_n
    int32_t n_prog;            // persistent programs G (<= n_tiles)
    int32_t group_m;           // tile-rows per band of the traversal order
};

// Slot of program p: programs that share an XCD get a contiguous range of
// slots, so the sub-tensors co-resident on one XCD's L2 are neighbours and
// share A row-blocks and B column-blocks.  A bijection of [0, G) when
// G % kXcds == 0; the identity otherwise.
__host__ __device__ inline int32_t program_slot(int32_t p, int32_t G) {
    if (G % kXcds != 0) return p;
    return (p % kXcds) * (G / kXcds) + p / kXcds;
}

// Linear traversal index t -> sub-tensor (tm, tn): bands of group_m
// tile-rows, column-major inside a band (the last band may be shorter).
// A bijection of [0, tiles_m * tiles_n).
__host__ __device__ inline void tile_coords(int32_t t, const Sched &s,
                                            int32_t &tm, int32_t &tn) {
    int32_t band_tiles = s.group_m * s.tiles_n;
    int32_t band = t / band_tiles;
    int32_t first_m = band * s.group_m;
    int32_t gm = s.tiles_m - first_m;
    if (gm > s.group_m) gm = s.group_m;
    int32_t in = t - band * band_tiles;
    tm = first_m + in % gm;
    tn = in / gm;
}

// Program p owns traversal indices program_slot(p) + r * G, r = 0, 1, ...
// below n_tiles.  tile_id(tm, tn) = tm * tiles_n + tn is the sub-tensor id
// used by tile_partition_check.

// Simple kernel: block of sub-tensors that program p of n_prog owns.  Blocks
// are numbered down the block columns (blocks_m per column), so that the
// programs of one XCD share columns of B.
__host__ __device__ inline void simple_block(int32_t p, int32_t n_prog,
                                             int32_t blocks_m, int32_t &bm,
                                             int32_t &bn) {
    const int32_t t = program_slot(p, n_prog);
    bm = t % blocks_m;
    bn = t / blocks_m;
}

// Simple kernel: leading K tiles of bk that a program loads without checks.
// All whole ones, except where a chunk of epc elements straddles column N of
// a B stored K x N (the program's columns start at n0, any multiple of the
// caller's partition, and it loads bn of them): such a chunk runs on into the
// next row, at most epc - 1 elements, so the tile with the last row, and
// rows shorter than a chunk, are left to the checked loads.
__host__ __device__ inline int32_t simple_whole_tiles(int32_t K, int32_t bk,
                                                      bool b_nk, int32_t N,
                                                      int32_t n0, int32_t bn,
                                                      int32_t epc) {
    if (b_nk || N - n0 >= bn || (N - n0) % epc == 0) return K / bk;
    return N >= epc && K > 0 ? (K - 1) / bk : 0;
}

// Simple kernel: does any chunk of an operand start inside a dword?  Rows are
// ld elements of es bytes apart; programs start at multiples of `step`
// elements of a row (0: all at its first, chunks along it are whole dwords).
inline bool simple_shift(uintptr_t base, int64_t ld, int64_t es,
                         int64_t step) {
    return ((base | (uint64_t)(ld * es) | (uint64_t)(step * es)) & 3) != 0;
}

// LDS stages of 128 x 128 sub-tensors where nothing else is named (0: the
// variant table's first, one program per compute unit).  Past one round of
// those, programs of two stages, two of them resident per compute unit: bf16
// 2304^3 (324) 38 us against 42 (K x N 37 against 49), 6000 x 1000 x 512 (376)
// 15.2 against 18.3 (14.8 against 19.0); e4m3 2304^3 20.4 against 27.5, 4096^3
// (1024) 69 against 85.  (bf16 stored N x K is up to a tenth ahead in one
// program at whole rounds of short K: 4096 x 2304 x 256 17.4 against 19.4.)
inline int rounds_128(int64_t tiles, int cus) {
    return tiles > (cus > 0 ? cus : 256) ? 2 : 0;
}

// The same for a grouped launch, whose sub-tensors differ in K: one program
// per compute unit runs the longest of them faster, two run more of them.
// `longest` and `sum`: K of the longest sub-tensor and of all together.
// bf16 by N x K (phased), 12 problems of 2048 x 2048 (3072 sub-tensors): even
// K 512 90 us against 79 with two stages, 2048 275 against 279, up to twice
// 2048 366 against 364; 20 of 512 x 512 (320), 2048 ... 4096 (1.26 times the
// mean at most) 44 against 55, 40 small ones, 256 ... 2560, 27 against 43.
// K x N: 12 of 2048 x 2048 x 512 103 us against 81, 40 of 512 x 512 (640), 2048
// ... 6144 (1.51) 141 against 128; but 20 (320) of those 67 against 86.
inline int grouped_stages_128(int64_t tiles, int64_t longest, int64_t sum,
                              bool b_nk, int cus) {
    if (cus <= 0) cus = 256;
    const bool two = b_nk ? sum <= 1024 * tiles && 4 * longest * tiles <=
                                                       5 * sum
                          : tiles > 2 * (int64_t)cus ||
                                10 * longest * tiles <= 13 * sum;
    return two ? rounds_128(tiles, cus) : 0;
}

// Kernel arguments of one tiled product.
struct GemmArgs {
    const void *a;
    const void *b;
    void *c;
    const float *scale_a;
    const float *scale_b;
    int32_t *wcount;
    int64_t lda, ldb, ldc;
    int32_t M, N, K;
    Sched s;
    // Products of planes: kp > 0 elements of K per plane, planes side by side
    // along K in A and B; product b (of K / kp) multiplies the planes that
    // four-bit field b of planes_a and planes_b names.
    int32_t kp = 0;
    uint32_t planes_a = 0, planes_b = 0;
};

// One problem of a grouped launch (device-side table entry).
struct GroupProblem {
    const void *a;
    const void *b;
    void *c;
    int64_t lda, ldb, ldc;
    int32_t M, N, K;
    int32_t tiles_m, tiles_n;
    int32_t tile_begin;  // prefix sum of tile counts, in table order
    int32_t c_bf16;      // output dtype: 0 f32, 1 bf16
    int32_t b_nk;        // B stored N x K
    int32_t *wcount;     // M x N store counters (ld N) or NULL
};

// Tiled kernel variants (compile-time instantiations), by index.
struct TiledVariant {
    int32_t dtype;   // tg_dtype of A and B
    int32_t bm, bn, bk, wm, wn;
    int32_t stages;  // LDS stages in the K-tile ring
    int32_t sched;   // tg_sched (lock-step or ping-pong)
    int32_t b_nk;
    int32_t c_bf16;
};

int tiled_variant_count();
const TiledVariant &tiled_variant(int i);
// Enqueue variant i; returns hipSuccess or the launch error.
hipError_t launch_tiled(int variant, const GemmArgs &args, hipStream_t st);
hipError_t launch_grouped(int variant, int n, int total_tiles, int n_prog,
                          const void *table_dev, hipStream_t st);
// The variant's kernel: variants of one kernel are names of the same launch.
const void *tiled_kernel(int variant);
// Whether variant i also runs products of planes (kp != 0).
bool tiled_planes(int variant);
int tiled_occupancy(int variant);  // resident workgroups per CU

// Skinny (decode-shaped) kernel.
struct SkinnyArgs {
    const void *x;       // M x K bf16 activations
    const void *w;       // N x K weights (bf16 or e4m3)
    void *y;             // M x N output
    const float *scale_a;
    const float *scale_w;  // per output column (row of W)
    int32_t *wcount;
    int64_t ldx, ldw, ldy;
    int32_t M, N, K;
    int32_t bn;          // output columns per program (16 or 32)
    // K split over programs: splitk programs share one sub-tensor's K, each
    // contracting the K steps [s * steps_per_split, (s + 1) *
    // steps_per_split) of its split s; with splitk > 1 they store their
    // partial tiles (unscaled binary32) into part[s][M][N] and, for the
    // fused normalisation, their rows' partial sums of squares into
    // ssq_part[s][M]; a merge launch then owns y.
    int32_t splitk;
    int32_t steps_per_split;
    float *part;
    float *ssq_part;
    // residual R (M x N, leading dimension ldr, bf16 when res_bf16) added
    // to every output before its one rounding, or nullptr
    const void *res;
    int64_t ldr;
    int32_t res_bf16;
};
// Streaming form of an unsplit product: the programs of bn columns that one
// workgroup runs, one after the other in the order of their columns; 0 where
// the plain form, a workgroup per program, is the faster or the only one.
int32_t skinny_stream(int w_dtype, int64_t M, int64_t N, int64_t K,
                      int64_t ldx, int64_t ldw, int32_t bn, int cus);
constexpr int kStreamRing = 4;   // tiles of the streaming form's LDS ring
// stream: skinny_stream's answer (0 with a K split).
hipError_t launch_skinny(int w_dtype, int c_bf16, int bn, int ksplit,
                         const SkinnyArgs &a, int stream, hipStream_t st);
// Merge of a split decode product: one program per bm x bn sub-tensor of
// y sums the splitk partial tiles in split order, applies the scales (and
// the fused normalisation's row scale when norm is set) and stores y.
hipError_t launch_skinny_merge(int c_bf16, const SkinnyArgs &a, bool norm,
                               float eps, hipStream_t st);

// Simple kernel: any dtype combination, any alignment.
struct SimpleArgs {
    const void *a;
    const void *b;
    void *c;
    const float *scale_a;
    const float *scale_b;
    int32_t *wcount;
    int64_t lda, ldb, ldc;
    int32_t M, N, K;
    int32_t a_dtype, b_dtype, c_bf16, b_nk;
    int32_t bm, bn;      // sub-tensor
    int32_t gm, gn;      // sub-tensors per program: gm bm and gn bn <= 128
    int32_t blocks_m;    // programs per block column
    int32_t n_prog;
};
// The same product of bf16 rows with e4m3 weights stored N x K, in programs
// of 2 x 2 sub-tensors of 64 x 64, on the phased 128 x 128 kernel.
hipError_t launch_mixed(const SimpleArgs &a, hipStream_t st);
hipError_t launch_simple(const SimpleArgs &a, hipStream_t st);

// Split of f32 operands into bf16 planes for the BF16xN precisions.
struct SplitArgs {
    const float *src;      // rows x cols
    uint16_t *dst;         // plane block b at b * plane_stride, rows ldd apart
    int64_t ld, ldd, plane_stride;
    int32_t rows, cols;
    int32_t blocks;        // nplanes blocks, block b = plane order[b]
    uint32_t order;        // four bits each
};
hipError_t launch_split(const SplitArgs &a, const SplitArgs &b,
                        hipStream_t st);

hipError_t launch_error_norm(const void *c, int c_bf16, const double *r,
                             int64_t n, double *out, hipStream_t st);

}  // namespace tg
