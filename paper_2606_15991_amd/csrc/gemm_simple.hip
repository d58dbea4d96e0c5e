// gemm_simple.hip -- tile programs for requests the tiled and decode kernels
// do not take: any dtype combination of the library, any leading dimension
// or alignment, any partition up to 64 x 64.
//
// One program owns a block of 1 x 1 or 2 x 2 neighbouring sub-tensors
// (simple_block in tg_internal.hpp) of at most BM x BN outputs and stores
// only into those.  bf16 and e4m3 operands are contracted by the 32x32x16
// bf16 matrix instruction (every e4m3 value is a bf16 value, so the decode
// is exact), binary32 operands by the 32x32x2 binary32 one; accumulation is
// binary32.
//
// K tiles are 128 bytes of LDS per row (64 bf16 or 32 binary32), double
// buffered; the next kDepth tiles are on their way from global memory into
// registers while one is contracted (one program of four wavefronts per
// SIMD group hides little latency by itself), then converted and stored to
// the other LDS buffer, one barrier per tile.  Global reads are 16 bytes per
// lane (8 of e4m3) from the dword below the chunk; where a chunk may start
// inside a dword (SHIFT: its row does, or for B stored K x N the partition's
// columns do) one more dword is read and the chunk shifted into place, since
// the unaligned access mode's own handling of such addresses takes about a
// cycle per lane (37.1 us with it, 21.7 with the shift at bf16 1111 x 1531 x
// 1003, B stored K x N).  No dword without a byte of the operand is touched.
// Direct-to-LDS loads need aligned rows and no conversion, so they stay with
// the tiled kernel.  The K tile with chunks that straddle the end of K (or,
// for B stored K x N, the operand's last row where chunks straddle N) is
// read element by element, first, while the other tiles' loads are in
// flight; rows and columns past the output repeat others or hold whatever
// follows, and are never stored.
//
// Bound: latency of the K-tile round (about 1.2 us at 1111 x 1531 x 1003:
// load, convert, store, barrier, contract) while programs are few, the
// matrix cores beyond.  Measured against the element-wise loads and
// binary32 FMAs from LDS that this kernel replaces: bf16 1111 x 1531 x 1003,
// 21.7 us against 467 (432 programs of 64 x 64).  bf16 rows by e4m3 weights:
// 512 x 5120 x 5120 with B stored K x N 47 us; stored N x K, where K is whole
// chunks of both, the mixed form of gemm_phased.hip takes it (44 us, 49 here).
// Three tiles in flight instead of two are no faster (22.6 us and, at those
// weights, 50: fewer wavefronts per SIMD), one is slower (62 us with 128 x 128
// blocks of four wavefronts).
#include "tg_device.hpp"
#include "tg_internal.hpp"

namespace tg {
namespace {

typedef __attribute__((address_space(3))) short lds_s16;
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int kRow = 128;             // LDS bytes of K per operand row
constexpr int kDepth = 2;              // K tiles in flight in registers

// Sources: bytes per element and per chunk of one 16-byte LDS chunk.
template <int DT>
struct Src {
    static constexpr int ES = DT == TG_F32 ? 4 : DT == TG_BF16 ? 2 : 1;
    static constexpr int EPC = DT == TG_F32 ? 4 : 8;   // elements per chunk
};

// The first n (0 .. EPC) elements of a chunk, zeros after them.
template <int DT>
__device__ __forceinline__ uint4 load_head(const char *p, int n) {
    constexpr int ES = Src<DT>::ES, EPC = Src<DT>::EPC;
    uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
    for (int e = 0; e < EPC; ++e)
        if (e < n) {
            uint32_t x;
            if constexpr (ES == 4) {
                __builtin_memcpy(&x, p + 4 * e, 4);
            } else if constexpr (ES == 2) {
                uint16_t h;
                __builtin_memcpy(&h, p + 2 * e, 2);
                x = h;
            } else {
                x = (uint8_t)p[e];
            }
            w[e * ES / 4] |= x << (8 * (e * ES % 4));
        }
    return uint4{w[0], w[1], w[2], w[3]};
}

// A chunk's dwords as they stand in LDS.
template <int DT>
__device__ __forceinline__ uint4 to_lds(const uint32_t *w) {
    if constexpr (DT == TG_FP8_E4M3) {
        const uint2 lo = e4m3x4_to_bf16x4(w[0]), hi = e4m3x4_to_bf16x4(w[1]);
        return uint4{lo.x, lo.y, hi.x, hi.y};
    } else {
        return uint4{w[0], w[1], w[2], w[3]};
    }
}

// K-tile barrier: LDS accesses complete, global loads stay in flight.
__device__ __forceinline__ void tile_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Row-major operand tile [rows][128 B]: chunk c of row r at c ^ ((r >> 1) &
// 7), free of bank conflicts for 16-byte reads of consecutive rows.
__device__ __forceinline__ int row_off(int r, int c) {
    return r * kRow + ((c ^ ((r >> 1) & 7)) << 4);
}

// k-major bf16 tile [64][BN]: chunk c of row k at c ^ f(k), so that the four
// rows of a transposing read land in distinct bank groups.
template <int BN>
__device__ __forceinline__ int kmaj_off(int k, int c) {
    constexpr int CPR = BN / 8;
    int f;
    if constexpr (CPR >= 16) {
        constexpr uint32_t tab = 0u | (4u << 8) | (10u << 16) | (14u << 24);
        f = (tab >> (8 * (k & 3))) & 0xff;
    } else {
        f = 2 * (k & 3);
    }
    return k * (BN * 2) + ((c ^ f) << 4);
}

// Eight k of column col0 + lane % 32 for the 32x32x16 instruction, from a
// k-major tile: two transposing reads.  In each 16-lane group lane r names
// row k = kb + r / 4 at columns c0 + 4 (r % 4) .. + 3 and lane i receives
// column c0 + i at rows kb .. kb + 3.
template <int BN>
__device__ __forceinline__ i32x4 read_kmaj(const char *Bs, int kk, int col0,
                                           int lane) {
    const int g = lane >> 4, r = lane & 15;
    const int n = col0 + (g & 1) * 16 + 4 * (r & 3);
    i32x4 out;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int k = kk * 16 + (g >> 1) * 8 + q * 4 + (r >> 2);
        const char *p = Bs + kmaj_off<BN>(k, n >> 3) + ((n & 7) << 1);
        const s16x4 v =
            __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p));
        const uint32_t v0 = (uint16_t)v[0], v1 = (uint16_t)v[1];
        const uint32_t v2 = (uint16_t)v[2], v3 = (uint16_t)v[3];
        out[2 * q] = (int)(v0 | (v1 << 16));
        out[2 * q + 1] = (int)(v2 | (v3 << 16));
    }
    return out;
}

// One operand's loader.  Row mode (A, and B stored N x K): LDS rows are
// operand rows, chunks run along K.  k-major mode (B stored K x N): LDS rows
// are k, chunks run along the columns.
template <int DT, bool KMAJ, int ROWS, bool SHIFT, int THREADS>
struct Loader {
    static constexpr int ES = Src<DT>::ES, EPC = Src<DT>::EPC;
    static constexpr int DW = ES * EPC / 4;            // dwords per chunk
    static constexpr int CPR = KMAJ ? ROWS / EPC : 8;  // chunks per LDS row
    static constexpr int N = ROWS * 8 / THREADS;      // chunks per thread
    static_assert(ROWS * 8 % THREADS == 0, "whole chunks per thread");
    // The chunks of K tile 0, from the dword that holds their first byte
    // (the tiles are whole dwords apart, so `mis` holds for all of them).
    const char *p[N];
    int mis[SHIFT ? N : 1];
    uint32_t v[kDepth][N][DW + (SHIFT ? 1 : 0)];

    // row0: first row (or column) of the block, rows: of the operand
    __device__ __forceinline__ void init(const void *base, int64_t ld,
                                         int row0, int rows, int tid) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int q = i * THREADS + tid, r = q / CPR, c = q % CPR;
            if constexpr (KMAJ) {
                const int col = row0 + c * EPC;
                p[i] = static_cast<const char *>(base) +
                       ((int64_t)r * ld + (col < rows ? col : 0)) * ES;
            } else {
                const int row = min(row0 + r, rows - 1);
                p[i] = static_cast<const char *>(base) +
                       ((int64_t)row * ld + c * EPC) * ES;
            }
            if constexpr (SHIFT) {
                mis[i] = (int)(reinterpret_cast<uintptr_t>(p[i]) & 3);
                p[i] -= mis[i];
            }
        }
    }
    __device__ __forceinline__ int64_t skip(int k0, int64_t ld) const {
        return (KMAJ ? (int64_t)k0 * ld : (int64_t)k0) * ES;
    }
    // K tile at k0, all of whose chunks lie inside the operand, into slot s
    __device__ __forceinline__ void load(int s, int k0, int64_t ld) {
        const int64_t o = skip(k0, ld);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const uint32_t *src = reinterpret_cast<const uint32_t *>(p[i] + o);
#pragma unroll
            for (int d = 0; d < DW; ++d) v[s][i][d] = src[d];
            if constexpr (SHIFT) v[s][i][DW] = src[mis[i] ? DW : DW - 1];
        }
    }
    __device__ __forceinline__ void store_chunk(char *lds, int i, int tid,
                                                const uint32_t *w) const {
        const int q = i * THREADS + tid, r = q / CPR, c = q % CPR;
        int off;
        if constexpr (!KMAJ) off = row_off(r, c);
        else if constexpr (DT == TG_F32) off = r * (ROWS * 4) + c * 16;
        else off = kmaj_off<ROWS>(r, c);
        st16(lds + off, to_lds<DT>(w));
    }
    __device__ __forceinline__ void store(int s, char *lds, int tid) const {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
            for (int d = 0; d < DW; ++d)
                w[d] = SHIFT ? __builtin_amdgcn_alignbyte(v[s][i][d + SHIFT],
                                                          v[s][i][d], mis[i])
                             : v[s][i][d];
            store_chunk(lds, i, tid, w);
        }
    }
    // K tile at k0 straight to LDS, every chunk checked against K and
    // (k-major) the columns
    __device__ __forceinline__ void copy_checked(char *lds, int k0, int K,
                                                 int64_t ld, int row0,
                                                 int rows, int tid) const {
        const int64_t o = skip(k0, ld);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int q = i * THREADS + tid, r = q / CPR, c = q % CPR;
            const int n = KMAJ ? (k0 + r < K ? rows - row0 - c * EPC : 0)
                               : K - k0 - c * EPC;
            const uint4 x =
                load_head<DT>(p[i] + (SHIFT ? mis[i] : 0) + o, n);
            const uint32_t w[4] = {x.x, x.y, x.z, x.w};
            store_chunk(lds, i, tid, w);
        }
    }
};

// Wavefronts along N of a block: 2 x 2 of them, 2 x 4 for 128 x 128.
constexpr int waves_n(int BM) { return BM > 64 ? 4 : 2; }

template <int ADT, int BDT, bool BNK, int BM, int BN, bool SHIFT>
__global__ __launch_bounds__(128 * waves_n(BM)) void gemm_simple_kernel(SimpleArgs g) {
    constexpr bool F32 = ADT == TG_F32;
    static_assert(F32 == (BDT == TG_F32), "binary32 pairs with itself");
    constexpr int BK = F32 ? 32 : 64;
    constexpr int WN = waves_n(BM), THREADS = 128 * WN;
    constexpr int TM = BM / 2, TN = BN / WN;
    constexpr int FM = TM / 32, FN = TN / 32;
    constexpr int STAGE = (BM + BN) * kRow;
    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int r = lane & 31, half = lane >> 5;
    int bm, bn;                                    // block of this program
    simple_block(blockIdx.x, gridDim.x, g.blocks_m, bm, bn);
    const int m0 = bm * g.gm * g.bm, n0 = bn * g.gn * g.bn;
    const int rows = min(g.gm * g.bm, g.M - m0);
    const int cols = min(g.gn * g.bn, g.N - n0);

    Loader<ADT, false, BM, SHIFT, THREADS> la;
    Loader<BDT, !BNK, BN, SHIFT, THREADS> lb;
    la.init(g.a, g.lda, m0, g.M, tid);
    lb.init(g.b, g.ldb, n0, g.N, tid);
    f32x16 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    auto contract = [&](const char *As) {
        const char *Bs = As + BM * kRow;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            i32x4 af[FM], bf[FN];
#pragma unroll
            for (int f = 0; f < FM; ++f)
                af[f] = *reinterpret_cast<const i32x4 *>(
                    As + row_off(wm * TM + f * 32 + r, 2 * kk + half));
#pragma unroll
            for (int f = 0; f < FN; ++f) {
                if constexpr (BNK) {
                    bf[f] = *reinterpret_cast<const i32x4 *>(
                        Bs + row_off(wn * TN + f * 32 + r, 2 * kk + half));
                } else if constexpr (F32) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        bf[f][e] = *reinterpret_cast<const int *>(
                            Bs + (8 * kk + 4 * half + e) * (BN * 4) +
                            (wn * TN + f * 32 + r) * 4);
                } else {
                    bf[f] = read_kmaj<BN>(Bs, kk, wn * TN + f * 32, lane);
                }
            }
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    if constexpr (F32) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const uint32_t ua = af[i][e], ub = bf[j][e];
                            acc[i][j] =
                                mfma_f32(as_f32(ua), as_f32(ub), acc[i][j]);
                        }
                    } else {
                        acc[i][j] = mfma_bf16(af[i], bf[j], acc[i][j]);
                    }
                }
        }
    };
    // tiles 0 .. nf - 1 load without checks
    const int nf = simple_whole_tiles(g.K, BK, BNK, g.N, n0, BN,
                                      Src<BDT>::EPC);
    auto load = [&](int s, int kt) {
        const int k0 = min(kt, nf - 1) * BK;   // past the last: unused
        la.load(s, k0, g.lda);
        lb.load(s, k0, g.ldb);
    };
    auto store = [&](int s, int kt) {
        char *st = smem + (kt & 1) * STAGE;
        la.store(s, st, tid);
        lb.store(s, st + BM * kRow, tid);
    };
    if (nf > 0) {
#pragma unroll
        for (int s = 0; s < kDepth; ++s) load(s, s);
    }
    for (int k0 = nf * BK; k0 < g.K; k0 += BK) {   // checked tiles
        char *st = smem + STAGE;
        la.copy_checked(st, k0, g.K, g.lda, m0, g.M, tid);
        lb.copy_checked(st + BM * kRow, k0, g.K, g.ldb, n0, g.N, tid);
        tile_barrier();
        contract(st);
        tile_barrier();
    }
    if (nf > 0) {
        store(0, 0);
        tile_barrier();
        auto step = [&](int kt, int s) {
            load(s, kt + kDepth);
            contract(smem + (kt & 1) * STAGE);
            store((s + 1) % kDepth, kt + 1);
            tile_barrier();
        };
        // (whole rounds without a branch, so that the compiler's load
        // counting waits for the oldest tile only)
        int kt = 0;
        for (; kt + kDepth <= nf; kt += kDepth) {
#pragma unroll
            for (int s = 0; s < kDepth; ++s) step(kt + s, s);
        }
#pragma unroll
        for (int s = 0; s < kDepth - 1; ++s)
            if (kt + s < nf) step(kt + s, s);
    }
    // 32 x 32 result layout: lane l, register v holds row 8 (v / 4) +
    // 4 (l / 32) + v % 4, column l % 32
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        const int c = wn * TN + j * 32 + r;
        if (c >= cols) continue;
        const int col = n0 + c;
        const float sb = g.scale_b ? g.scale_b[col] : 1.f;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int q = wm * TM + i * 32 + 8 * (v >> 2) + 4 * half +
                              (v & 3);
                if (q >= rows) continue;
                const int row = m0 + q;
                float x = acc[i][j][v];
                if (g.scale_a) x *= g.scale_a[row];
                if (g.scale_b) x *= sb;
                const int64_t off = (int64_t)row * g.ldc + col;
                if (g.c_bf16)
                    static_cast<uint16_t *>(g.c)[off] = f32_to_bf16_bits(x);
                else
                    static_cast<float *>(g.c)[off] = x;
                if (g.wcount)
                    atomicAdd(&g.wcount[(int64_t)row * g.N + col], 1);
            }
    }
}

template <int ADT, int BDT, bool BNK, int BM, int BN, bool SHIFT>
hipError_t launch_block(const SimpleArgs &a, hipStream_t st) {
    constexpr int smem = 2 * (BM + BN) * kRow;
    static_assert(smem <= 65536, "LDS without opting in");
    hipLaunchKernelGGL((gemm_simple_kernel<ADT, BDT, BNK, BM, BN, SHIFT>),
                       dim3(a.n_prog), dim3(128 * waves_n(BM)), smem, st, a);
    return hipGetLastError();
}

template <int ADT, int BDT, bool BNK, bool SHIFT>
hipError_t launch_blocks(const SimpleArgs &a, hipStream_t st) {
    return a.gm * a.bm > 64 || a.gn * a.bn > 64
               ? launch_block<ADT, BDT, BNK, 128, 128, SHIFT>(a, st)
               : launch_block<ADT, BDT, BNK, 64, 64, SHIFT>(a, st);
}

template <int ADT, int BDT>
hipError_t launch_layout(const SimpleArgs &a, hipStream_t st) {
    const bool sh =
        simple_shift(reinterpret_cast<uintptr_t>(a.a), a.lda, Src<ADT>::ES,
                     0) ||
        simple_shift(reinterpret_cast<uintptr_t>(a.b), a.ldb, Src<BDT>::ES,
                     a.b_nk ? 0 : a.gn * a.bn);
    if (a.b_nk)
        return sh ? launch_blocks<ADT, BDT, true, true>(a, st)
                  : launch_blocks<ADT, BDT, true, false>(a, st);
    return sh ? launch_blocks<ADT, BDT, false, true>(a, st)
              : launch_blocks<ADT, BDT, false, false>(a, st);
}

}  // namespace

hipError_t launch_simple(const SimpleArgs &a, hipStream_t st) {
    if (a.bm < 1 || a.bn < 1 || a.gm * a.bm > 128 || a.gn * a.bn > 128)
        return hipErrorInvalidValue;
    if (a.a_dtype == TG_F32 && a.b_dtype == TG_F32)
        return launch_layout<TG_F32, TG_F32>(a, st);
    if (a.a_dtype == TG_BF16 && a.b_dtype == TG_BF16)
        return launch_layout<TG_BF16, TG_BF16>(a, st);
    if (a.a_dtype == TG_BF16 && a.b_dtype == TG_FP8_E4M3)
        return launch_layout<TG_BF16, TG_FP8_E4M3>(a, st);
    if (a.a_dtype == TG_FP8_E4M3 && a.b_dtype == TG_FP8_E4M3)
        return launch_layout<TG_FP8_E4M3, TG_FP8_E4M3>(a, st);
    return hipErrorInvalidValue;
}

}  // namespace tg
