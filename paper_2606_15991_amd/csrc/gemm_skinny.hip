// gemm_skinny.hip -- decode-shaped products y[M x N] = x[M x K] . W^T with
// M <= 16 and W stored N x K (bf16, or OCP E4M3 with one fp32 scale per row
// of W, i.e. per output column).
//
// The work is bound by streaming W from HBM once (arithmetic intensity about
// M flop per weight byte).  One tile program owns bn <= 16 RT output columns
// (RT row tiles of 16 weight rows, the rows past its bn repeating its last
// row) for all M rows, so that bn can divide N into a whole number of
// programs per compute unit; its KS wavefronts split
// K between them and stream their share of the weight rows with 16-byte
// loads, several in flight per lane.  With two row tiles every activation
// chunk loaded serves two weight chunks.  The contraction runs on the 16x16x32 bf16 matrix
// instruction with the weight rows as the A operand and the (zero-padded)
// activation rows as the B operand; E4M3 weights are decoded exactly to
// bf16 in registers first (there is no mixed bf16 x e4m3 matrix
// instruction).  The KS partial tiles are summed in LDS in a fixed order,
// and one wavefront stores the sub-tensor: deterministic, no atomics.
//
// Where one program per sub-tensor leaves compute units idle (few output
// columns) or streams too few bytes at once (long rows), the K steps are
// also split over `splitk` programs per sub-tensor (grid y).  Each stores
// its partial tile, unscaled, into its own slice part[s][M][N] of a
// workspace partitioned by (split, sub-tensor); a second launch, whose
// program p owns sub-tensor p of y, sums the slices in split order and
// stores y.  No atomics: the result is the same on every run.
#include "tg_device.hpp"
#include "tg_elementwise.hpp"
#include "tg_internal.hpp"
#include "tg_tiled.hpp"

namespace tg {
namespace {


// 16 bytes at p of which only the first n (0..16) are inside the operand;
// the rest read as zero.  Used for the one chunk per row that straddles K.
__device__ __forceinline__ uint4 ld16_head(const char *p, int n) {
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int b = 0; b < 16; ++b)
        if (b < n) w[b >> 2] |= (uint32_t)(uint8_t)p[b] << (8 * (b & 3));
    return uint4{w[0], w[1], w[2], w[3]};
}

// Chunk of `epc` elements of `es` bytes starting at element k of a row of
// `K` elements: whole, partial, or past the end.
__device__ __forceinline__ uint4 ld_chunk(const char *row, int k, int K,
                                          int epc, int es) {
    if (k + epc <= K) return ld16(row + (int64_t)k * es);
    if (k < K) return ld16_head(row + (int64_t)k * es, (K - k) * es);
    return uint4{0, 0, 0, 0};
}

// Residual element (m, n), as binary32.
__device__ __forceinline__ float residual_at(const SkinnyArgs &g, int m,
                                             int n) {
    const int64_t off = (int64_t)m * g.ldr + n;
    return g.res_bf16
               ? bf16_bits_to_f32(static_cast<const uint16_t *>(g.res)[off])
               : static_cast<const float *>(g.res)[off];
}

// NORM (1 or 2): the activation rows are RMS-normalised on the fly (the
// normalisation step of the decode layer fused into the product): each
// activation chunk is multiplied by the matching chunk of the normalisation
// weights nw and rounded to bf16 before the contraction, the lanes
// accumulate the squares of the raw activations, and every output of row m
// is multiplied by 1 / sqrt(mean_k x[m, k]^2 + eps).  Every activation
// element of a row is loaded by exactly one lane of one wavefront of the
// program, so the program holds the whole row's sum of squares after its
// reduction.  NORM = 2 first copies the program's slice of nw into LDS and
// reads each chunk from there when it is needed; NORM = 1 (slices longer
// than the LDS budget) loads nw chunks into registers beside the
// activation chunks, which costs a third more registers per lane.
template <int WDT, int KS, bool CBF16, int RT, int NORM>
__device__ __forceinline__ void skinny_body(const SkinnyArgs &g,
                                            const void *nw, float eps) {
    // Elements of K covered by one 16-byte weight load per lane group:
    // bf16: 8 per lane, 4 lane groups -> 32;  e4m3: 16 per lane -> 64.
    constexpr int EPL = WDT == TG_BF16 ? 8 : 16;
    constexpr int KSTEP = 4 * EPL;
    // K steps per super-step: eight weight loads per lane either way
    constexpr int UNROLL = 8 / RT;
    __shared__ f32x4 part[KS][RT][64];
    __shared__ float ssq[NORM ? KS : 1][64];
    extern __shared__ uint4 nw_lds[];   // NORM == 2: this program's nw

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n0 = blockIdx.x * g.bn;
    const int n_end = min(n0 + g.bn, g.N);   // this program's columns
    const int r = lane & 15, grp = lane >> 4;
    const bool xrow_ok = r < g.M;
    const int xrow = xrow_ok ? r : 0;

    const char *W[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        int wrow = n0 + 16 * t + r;
        wrow = wrow < n_end ? wrow : n_end - 1;
        W[t] = static_cast<const char *>(g.w) +
               (int64_t)wrow * g.ldw * (WDT == TG_BF16 ? 2 : 1);
    }
    const uint16_t *X = static_cast<const uint16_t *>(g.x) +
                        (int64_t)xrow * g.ldx;

    f32x4 acc[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int nsteps = (g.K + KSTEP - 1) / KSTEP;
    // this program's K steps: [sb, se) (the whole of K without a split)
    const int sb = blockIdx.y * g.steps_per_split;
    const int se = min(nsteps, sb + g.steps_per_split);
    constexpr int WES = WDT == TG_BF16 ? 2 : 1;
    constexpr int XV = WDT == TG_BF16 ? 1 : 2;   // activation chunks per step
    const char *Xc = reinterpret_cast<const char *>(X);
    const char *NWc = static_cast<const char *>(nw);
    float ss = 0.f;
    // Wave w takes super-steps w, w + KS, ... of UNROLL K steps each: all
    // UNROLL weight and activation chunks of a super-step are loaded before
    // any is contracted, so every lane has UNROLL weight loads in flight
    // (the other wavefronts of the SIMD overlap their own).  Super-steps
    // wholly inside K load without bounds tests: rows beyond the program's
    // columns were clamped to its last row (the repeated loads hit the same
    // cache lines) and activation rows beyond M read row 0, and both only
    // feed outputs that are never stored.  A ragged K tail takes the checked
    // loads.
    // Two register buffers (the wave's next super-step is loaded while the
    // current one is contracted) where the register budget allows: up to
    // 512 threads per program.
    constexpr int NB = KS <= 8 ? 2 : 1;
    uint4 wv[NB][UNROLL][RT], xv[NB][UNROLL][XV];
    uint4 nv[NORM == 1 ? NB : 1][NORM == 1 ? UNROLL : 1][NORM == 1 ? XV : 1];
    const int kb = sb * KSTEP;   // first element of this program's K range
    int s0 = 0;                  // first K step of the buffer contracted
    // NORM == 2: nw[kb, kb + (se - sb) KSTEP) into LDS as 16-byte chunks,
    // zeros past K, up to the end of the last super-step (its steps past se
    // multiply zero activations with what stands here: a leftover NaN or
    // infinity would not vanish); run after the first weight loads are
    // issued, so that its round trip overlaps theirs
    auto stage_nw = [&]() {
        if constexpr (NORM == 2) {
            const int chunks =
                (se - sb + UNROLL - 1) / UNROLL * UNROLL * KSTEP / 8;
            for (int i = threadIdx.x; i < chunks; i += KS * 64)
                nw_lds[i] = ld_chunk(NWc, kb + 8 * i, g.K, 8, 2);
            __syncthreads();
        }
    };
    auto load_fast = [&](int s0, int b) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int k = (s0 + u) * KSTEP + grp * EPL;
#pragma unroll
            for (int t = 0; t < RT; ++t)
                wv[b][u][t] = ld16(W[t] + (int64_t)k * WES);
#pragma unroll
            for (int c = 0; c < XV; ++c) {
                xv[b][u][c] = ld16(Xc + (int64_t)(k + 8 * c) * 2);
                if constexpr (NORM == 1)
                    nv[b][u][c] = ld16(NWc + (int64_t)(k + 8 * c) * 2);
            }
        }
    };
    auto load_checked = [&](int s0, int b) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int k = (s0 + u) * KSTEP + grp * EPL;
            const bool live = s0 + u < se;
#pragma unroll
            for (int t = 0; t < RT; ++t)
                wv[b][u][t] = live ? ld_chunk(W[t], k, g.K, EPL, WES)
                                   : uint4{0, 0, 0, 0};
            const bool ok = live && k < g.K;
#pragma unroll
            for (int c = 0; c < XV; ++c) {
                xv[b][u][c] = ok ? ld_chunk(Xc, k + 8 * c, g.K, 8, 2)
                                 : uint4{0, 0, 0, 0};
                if constexpr (NORM == 1)
                    nv[b][u][c] = ok ? ld_chunk(NWc, k + 8 * c, g.K, 8, 2)
                                     : uint4{0, 0, 0, 0};
            }
        }
    };
    // x * nw rounded to bf16 (round to nearest even, by the packed
    // hardware conversion), eight at a time; squares of x into ss
    auto normed = [&](const uint4 &x, const uint4 &w) -> uint4 {
        typedef float f32x2_t __attribute__((ext_vector_type(2)));
        typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
        const uint32_t xa[4] = {x.x, x.y, x.z, x.w};
        const uint32_t wa[4] = {w.x, w.y, w.z, w.w};
        uint32_t o[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float xl = __uint_as_float(xa[q] << 16);
            const float xh = __uint_as_float(xa[q] & 0xffff0000u);
            ss += xl * xl;
            ss += xh * xh;
            const f32x2_t p = {xl * __uint_as_float(wa[q] << 16),
                               xh * __uint_as_float(wa[q] & 0xffff0000u)};
            o[q] = __builtin_bit_cast(
                uint32_t, __builtin_convertvector(p, bf16x2_t));
        }
        return uint4{o[0], o[1], o[2], o[3]};
    };
    // buffer b holds the K steps s0 .. s0 + UNROLL - 1 (s0 as it stands
    // at every call below)
    auto contract = [&](int b) {
        if constexpr (NORM == 1) {
#pragma unroll
            for (int u = 0; u < UNROLL; ++u)
#pragma unroll
                for (int c = 0; c < XV; ++c)
                    xv[b][u][c] = normed(xv[b][u][c], nv[b][u][c]);
        } else if constexpr (NORM == 2) {
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const int k = (s0 + u) * KSTEP + grp * EPL;
#pragma unroll
                for (int c = 0; c < XV; ++c)
                    xv[b][u][c] = normed(xv[b][u][c],
                                         nw_lds[(k - kb) / 8 + c]);
            }
        }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u)
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                if constexpr (WDT == TG_BF16) {
                    acc[t] = mfma16_bf16(
                        __builtin_bit_cast(i32x4, wv[b][u][t]),
                        __builtin_bit_cast(i32x4, xv[b][u][0]), acc[t]);
                } else {
                    uint2 w01 = e4m3x4_to_bf16x4(wv[b][u][t].x);
                    uint2 w23 = e4m3x4_to_bf16x4(wv[b][u][t].y);
                    uint2 w45 = e4m3x4_to_bf16x4(wv[b][u][t].z);
                    uint2 w67 = e4m3x4_to_bf16x4(wv[b][u][t].w);
                    i32x4 wa = {(int)w01.x, (int)w01.y, (int)w23.x, (int)w23.y};
                    i32x4 wb = {(int)w45.x, (int)w45.y, (int)w67.x, (int)w67.y};
                    acc[t] = mfma16_bf16(
                        wa, __builtin_bit_cast(i32x4, xv[b][u][0]), acc[t]);
                    acc[t] = mfma16_bf16(
                        wb, __builtin_bit_cast(i32x4, xv[b][u][1]), acc[t]);
                }
            }
    };
    constexpr int STRIDE = KS * UNROLL;
    // steps of this program wholly inside K (split boundaries fall on
    // super-step boundaries, so only the last split has a ragged tail)
    const int nfull = min(g.K / KSTEP, se);
    s0 = sb + wave * UNROLL;
    if constexpr (NB == 2) {
        bool have0 = s0 + UNROLL <= nfull;
        if (have0) load_fast(s0, 0);
        stage_nw();
        while (have0) {
            const int s1 = s0 + STRIDE;
            const bool have1 = s1 + UNROLL <= nfull;
            if (have1) load_fast(s1, NB - 1);
            contract(0);
            s0 = s1;
            if (!have1) break;
            const int s2 = s1 + STRIDE;
            have0 = s2 + UNROLL <= nfull;
            if (have0) load_fast(s2, 0);
            contract(NB - 1);
            s0 = s2;
        }
    } else {
        stage_nw();
        for (; s0 + UNROLL <= nfull; s0 += STRIDE) {
            load_fast(s0, 0);
            contract(0);
        }
    }
    for (; s0 < se; s0 += STRIDE) {           // ragged tail, bounds checked
        load_checked(s0, 0);
        contract(0);
    }

#pragma unroll
    for (int t = 0; t < RT; ++t) part[wave][t][lane] = acc[t];
    if constexpr (NORM) ssq[wave][lane] = ss;
    __syncthreads();
    if (wave != 0) return;
    // 16 x 16 result layout: lane l, register v holds row 4 * (l / 16) + v
    // (a weight row, i.e. output column) and column l % 16 (an output row).
    const int m = lane & 15;
    if (m >= g.M) return;
    if (g.splitk > 1) {
        // partial tile of split blockIdx.y, unscaled, into its own slice
        float *dst = g.part + (int64_t)blockIdx.y * g.M * g.N +
                     (int64_t)m * g.N;
        if constexpr (NORM) {
            if (blockIdx.x == 0 && grp == 0) {
                float tot = 0.f;
#pragma unroll
                for (int w = 0; w < KS; ++w)
#pragma unroll
                    for (int q = 0; q < 4; ++q) tot += ssq[w][m + 16 * q];
                g.ssq_part[blockIdx.y * g.M + m] = tot;
            }
        }
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            f32x4 s = part[0][t][lane];
#pragma unroll
            for (int w = 1; w < KS; ++w) {
                f32x4 p = part[w][t][lane];
                s[0] += p[0]; s[1] += p[1]; s[2] += p[2]; s[3] += p[3];
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int n = n0 + 16 * t + 4 * grp + v;
                if (n < n_end) dst[n] = s[v];
            }
        }
        return;
    }
    float sa = g.scale_a ? g.scale_a[m] : 1.0f;
    if constexpr (NORM) {
        // row m's squares sit in lanes m, m + 16, m + 32, m + 48 of every
        // wavefront; summed in a fixed order
        float tot = 0.f;
#pragma unroll
        for (int w = 0; w < KS; ++w)
#pragma unroll
            for (int q = 0; q < 4; ++q) tot += ssq[w][m + 16 * q];
        sa *= 1.0f / sqrtf(tot / (float)g.K + eps);
    }
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        f32x4 s = part[0][t][lane];
#pragma unroll
        for (int w = 1; w < KS; ++w) {
            f32x4 p = part[w][t][lane];
            s[0] += p[0]; s[1] += p[1]; s[2] += p[2]; s[3] += p[3];
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int n = n0 + 16 * t + 4 * grp + v;
            if (n < n_end) {
                float y = s[v] * sa;
                if (g.scale_w) y *= g.scale_w[n];
                if (g.res) y += residual_at(g, m, n);
                int64_t off = (int64_t)m * g.ldy + n;
                if constexpr (CBF16)
                    static_cast<uint16_t *>(g.y)[off] = f32_to_bf16_bits(y);
                else
                    static_cast<float *>(g.y)[off] = y;
                if (g.wcount) atomicAdd(&g.wcount[(int64_t)m * g.N + n], 1);
            }
        }
    }
}

template <int WDT, int KS, bool CBF16, int RT>
__global__ __launch_bounds__(KS * 64) void gemm_skinny_kernel(SkinnyArgs g) {
    skinny_body<WDT, KS, CBF16, RT, 0>(g, nullptr, 0.f);
}

// (bf16 weights, staged nw: three wavefronts per SIMD, as the plain bf16
// product runs; the staged variant fits the register budget for it)
template <int WDT, int KS, bool CBF16, int RT, int NORM>
__global__ __launch_bounds__(KS * 64) __attribute__((amdgpu_waves_per_eu(
    NORM == 2 && WDT == TG_BF16 ? 3 : 1))) void gemm_skinny_norm_kernel(
    SkinnyNormArgs a) {
    skinny_body<WDT, KS, CBF16, RT, NORM>(a.s, a.norm_w, a.eps);
}

// Merge of a split product: program p owns sub-tensor p of y (M rows x bn
// columns); its threads take the sub-tensor's elements in row-major order
// and sum the splitk partial values of each in split order, then apply the
// scales and add the residual.
template <bool CBF16, bool NORM>
__global__ __launch_bounds__(256) void skinny_merge_kernel(SkinnyArgs g,
                                                           float eps) {
    const int n0 = blockIdx.x * g.bn;
    for (int e = threadIdx.x; e < g.M * g.bn; e += 256) {
        const int m = e / g.bn, n = n0 + e % g.bn;
        if (n >= g.N) continue;
        const float *src = g.part + (int64_t)m * g.N + n;
        const int64_t slice = (int64_t)g.M * g.N;
        float v = src[0];
        for (int s = 1; s < g.splitk; ++s) v += src[s * slice];
        float sa = g.scale_a ? g.scale_a[m] : 1.0f;
        if constexpr (NORM) {
            float tot = g.ssq_part[m];
            for (int s = 1; s < g.splitk; ++s) tot += g.ssq_part[s * g.M + m];
            sa *= 1.0f / sqrtf(tot / (float)g.K + eps);
        }
        float y = v * sa;
        if (g.scale_w) y *= g.scale_w[n];
        if (g.res) y += residual_at(g, m, n);
        const int64_t off = (int64_t)m * g.ldy + n;
        if constexpr (CBF16)
            static_cast<uint16_t *>(g.y)[off] = f32_to_bf16_bits(y);
        else
            static_cast<float *>(g.y)[off] = y;
        if (g.wcount) atomicAdd(&g.wcount[(int64_t)m * g.N + n], 1);
    }
}

// Streaming form of the unsplit product for outputs of many columns.  What
// holds the plain form back is the load path: a fragment load touches 16
// rows of 64 bytes, 64 cache-line lookups for 1 KiB, and each program of few
// columns loads the activations anew, as many bytes as weights.  Here a
// workgroup of eight wavefronts takes `q` consecutive programs, i.e. a run
// of q bn columns in row tiles of 16 whatever bn is.  The wavefronts share
// K, 128 bytes of every row in turn.  Weights go from memory to LDS by
// direct loads of whole lines (8 rows of 128 bytes; the 16-byte chunk c of
// row r at c ^ ((r >> 1) & 7) against bank conflicts, of which 37 % of the
// LDS cycles are left; wavefronts wait for memory 65 % of their time) into a
// ring of kStreamRing tiles per wavefront, which no other
// wavefront reads: no barrier, and the next kStreamRing - 1 tiles in flight
// throughout, over the end of a row tile too.  The activations stand in LDS
// once.  At the end of a row tile the
// wavefronts' partial tiles meet in LDS and are summed in their order.
// Measured (cold weights): e4m3 (8, 51200, 5120) 53 us against 73, one row
// 47 against 58; bf16 98 against 118 and 92 against 100; (1, 5120, 5120) e4m3
// 9.0 against 9.8; reading 262 MB alone takes 45 us on this chip.
constexpr int kStreamWaves = 8;
constexpr int kStreamTile = 16 * 128;                       // bytes
constexpr int kStreamLds =    // ring, and two sets of partial tiles
    kStreamWaves * (kStreamRing * kStreamTile + 2 * 1024);

template <int WDT, bool CBF16>
__global__ __launch_bounds__(kStreamWaves * 64) void skinny_stream_kernel(
    SkinnyArgs g, int q) {
    constexpr int WES = WDT == TG_BF16 ? 2 : 1, XV = WDT == TG_BF16 ? 1 : 2;
    extern __shared__ __align__(1024) char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    char *ring = lds + wave * kStreamRing * kStreamTile;
    float *part = reinterpret_cast<float *>(
        lds + kStreamWaves * kStreamRing * kStreamTile);
    char *xs = lds + kStreamLds;
    const int r = lane & 15, grp = lane >> 4;
    // this workgroup's columns
    const int c0 = blockIdx.x * q * g.bn;
    const int cols = min(g.N - c0, q * g.bn);
    const int tiles = (cols + 15) / 16;
    const int kbytes = g.K * WES, nkb = (kbytes + 127) / 128;
    const uint32_t ldw = (uint32_t)(g.ldw * WES);
    // rows past the columns lie past the buffer's end and load as zeros
    const i32x4 W = make_srd(
        static_cast<const char *>(g.w) + (int64_t)c0 * g.ldw * WES,
        (uint32_t)cols * ldw);
    // this lane's row and chunk of both loads of a tile
    const int lrow = lane >> 3;
    uint32_t lch[2], loff[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = i * 8 + lrow;
        lch[i] = ((lane & 7) ^ ((row >> 1) & 7)) * 16;
        loff[i] = row * ldw + lch[i];
    }
    // The wavefront's tiles in order: 128-byte blocks wave, wave + 8, ... of
    // row tile 0, of row tile 1 and so on.
    const int total =
        tiles * ((nkb - wave + kStreamWaves - 1) / kStreamWaves);
    int ikb = wave;               // block of the tile that is loaded next
    uint32_t irow = 0;            // byte offset of its rows
    auto issue = [&](int slot) {
        char *dst = ring + slot * kStreamTile;
        const uint32_t k = ikb * 128;
        const bool whole = (ikb + 1) * 128 <= kbytes;
        uint32_t v[2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
            v[i] = whole || (int)(k + lch[i]) < kbytes
                       ? irow + loff[i] + k : kOutOfRange;
        dma16<true>(W, dst, v[0]);
        dma16<false>(W, dst + 1024, v[1]);
        ikb += kStreamWaves;
        if (ikb >= nkb) {
            ikb = wave;
            irow += 16 * ldw;
        }
    };
#pragma unroll
    for (int i = 0; i < kStreamRing; ++i)
        if (i < total) issue(i);
    // Activations: 16-byte chunk kc of row m at chunk kc ^ m of its row, rows
    // of whole 256 bytes, zeros past K.  (Direct loads: all of them are in
    // flight at once; through registers, row by row, 80 KiB took 9 us.)
    const int rowc = (g.K + 127) / 128 * 16;     // chunks of a row
    {
        const i32x4 X = make_srd(g.x, (uint32_t)(g.M * g.ldx * 2));
        for (int i = wave; i * 64 < g.M * rowc; i += kStreamWaves) {
            const int e = i * 64 + lane, m = e / rowc;
            const int kc = (e - m * rowc) ^ m;
            dma16<true>(X, xs + i * 1024,
                        m < g.M && kc * 8 < g.K
                            ? (uint32_t)(m * g.ldx * 2 + kc * 16)
                            : kOutOfRange);
        }
        wait_vmem();
        __syncthreads();
    }
    const int wr0 = r * 128 + ((grp ^ ((r >> 1) & 7)) << 4);
    const int wr1 = r * 128 + (((grp + 4) ^ ((r >> 1) & 7)) << 4);
    // activation chunks of block kb: bf16 kb * 8 + 4 h + grp, e4m3 kb * 16 +
    // 8 h + 2 grp + c; this wavefront's blocks are all even or all odd
    const int xrow = r < g.M ? r : 0;
    const char *xp[2 * XV];
#pragma unroll
    for (int c = 0; c < 2 * XV; ++c) {
        const int kc = XV == 1 ? (wave & 1) * 8 + 4 * c + grp
                               : 8 * (c >> 1) + 2 * grp + (c & 1);
        xp[c] = xs + (xrow * rowc + (kc ^ xrow)) * 16;
    }
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    int kb = wave, tile = 0;
    for (int it = 0; it < total; ++it) {
        if (total - 1 - it >= kStreamRing - 1)
            wait_vmem_le<2 * (kStreamRing - 1)>();
        else
            wait_vmem();
        asm volatile("" ::: "memory");
        const int slot = it % kStreamRing;
        const char *wt = ring + slot * kStreamTile;
        const i32x4 w[2] = {*reinterpret_cast<const i32x4 *>(wt + wr0),
                            *reinterpret_cast<const i32x4 *>(wt + wr1)};
        i32x4 x[2 * XV];
        const int xk = (XV == 1 ? kb >> 1 : kb) * 256;
#pragma unroll
        for (int c = 0; c < 2 * XV; ++c)
            x[c] = *reinterpret_cast<const i32x4 *>(xp[c] + xk);
        // the slot is free once its fragments are in registers
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (it + kStreamRing < total) issue(slot);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if constexpr (WDT == TG_BF16) {
                acc = mfma16_bf16(w[h], x[h], acc);
            } else {
                const uint2 w0 = e4m3x4_to_bf16x4(w[h][0]);
                const uint2 w1 = e4m3x4_to_bf16x4(w[h][1]);
                const uint2 w2 = e4m3x4_to_bf16x4(w[h][2]);
                const uint2 w3 = e4m3x4_to_bf16x4(w[h][3]);
                acc = mfma16_bf16(i32x4{(int)w0.x, (int)w0.y, (int)w1.x,
                                        (int)w1.y}, x[XV * h], acc);
                acc = mfma16_bf16(i32x4{(int)w2.x, (int)w2.y, (int)w3.x,
                                        (int)w3.y}, x[XV * h + XV - 1], acc);
            }
        }
        kb += kStreamWaves;
        if (kb < nkb) continue;
        // The end of a row tile.  The set of partial tiles written now was
        // last read before the barrier of the row tile before.
        kb = wave;
        float *set = part + (tile & 1) * kStreamWaves * 256;
        reinterpret_cast<f32x4 *>(set)[wave * 64 + lane] = acc;
        acc = f32x4{0.f, 0.f, 0.f, 0.f};
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        // four wavefronts in turn: thread e: lane e / 4, register e % 4 of
        // the result layout (lane l, register v: weight row 4 (l / 16) + v,
        // output row l % 16)
        const int m = (tid >> 2) & 15, e = tid & 255;
        const int c = tile * 16 + 4 * (e >> 6) + (e & 3);
        if ((wave >> 2) == (tile & 1) && m < g.M && c < cols) {
            float s = set[e];
#pragma unroll
            for (int w = 1; w < kStreamWaves; ++w) s += set[w * 256 + e];
            const int n = c0 + c;
            float y = s * (g.scale_a ? g.scale_a[m] : 1.0f);
            if (g.scale_w) y *= g.scale_w[n];
            if (g.res) y += residual_at(g, m, n);
            const int64_t off = (int64_t)m * g.ldy + n;
            if constexpr (CBF16)
                static_cast<uint16_t *>(g.y)[off] = f32_to_bf16_bits(y);
            else
                static_cast<float *>(g.y)[off] = y;
            if (g.wcount) atomicAdd(&g.wcount[(int64_t)m * g.N + n], 1);
        }
        ++tile;
    }
}

// Bytes of LDS of the streaming form, or 0 where it cannot run the product:
// K of whole 16-byte weight chunks, a block of K for every wavefront, the
// activations within LDS.
int64_t stream_lds(int64_t kbytes, int64_t M, int64_t K, int64_t ldx) {
    const int64_t nkb = (kbytes + 127) / 128;
    if (kbytes % 16 || kbytes > 0x7fffffff || nkb < kStreamWaves) return 0;
    const int64_t x = (K + 127) / 128 * 256 * M;
    const int64_t lds = kStreamLds + (x + 1023) / 1024 * 1024;
    return lds <= 160 * 1024 && M * ldx * 2 < 0x7fffffff ? lds : 0;
}

// Whether the streaming form is the faster one (cold weights, blocks of 128
// bytes of K).  Its workgroups are dealt whole programs, so the last ones may
// get none: from 85 in 100 workgroups' worth of programs on it is ahead (e4m3,
// one row: (25600, 5120) in 16-column programs, 89 in 100, 28.4 us against
// 34.9, but (10240, 5120), 83, 18.7 against 17.7 and (12800, 5120), 78, 21.8
// against 21.0).  And a row tile ends in a barrier, which needs K to be
// hidden:
//  * twelve blocks: e4m3 (4, 51200, 1024), eight, 19.7 us against 16.8, (4,
//    30000, 1536), twelve, 15.5 against 16.3;
//  * more where the plain form has no half-used row tiles and few rows of
//    activations to load (up to four, programs of up to 16 columns) and the
//    streaming one several programs a workgroup.  bf16 with one or two rows:
//    25 ((1, 51200, 1024), 16 blocks, 21.1 against 19.4, 1536, 24, 29.5 against
//    27.8, 2048, 32, 1.04 times as fast), only where the blocks go round the
//    eight wavefronts more than nine tenths evenly ((1, 23008, 2112), 33, 20.4
//    against 19.1, (1, 20224, 1648), 26, 15.0 against 14.2), and 65 where rows
//    are no whole 128 bytes, so that every block lies on two lines ((1, 33872,
//    1808), 29, 28.5 against 23.8, (2, 25856, 2976), 47, 30.9 against 29.2, past
//    80 level).  bf16 with three or four rows: 17 ((4, 16384, 1024), 16, 9.3
//    against 9.0, 1280, 20, 1.03 times as fast).  e4m3 with one or two rows and
//    up to five programs a workgroup: 17 ((1, 16384, 2048), 16, 10.6 against
//    9.9, 2304, 18, 1.05 times as fast; (1, 23337, 2048) in six 1.05 times);
//  * such bf16 products in two programs a workgroup not where workgroups start
//    a multiple of 256 KiB apart and so read the same channels of memory side
//    by side: (1, 8192, 4096) 16.4 us against 15.7, (1, 8192, 8192) 31.1
//    against 29.0, (4, 8192, 8192) 31.5 against 29.8, while K = 5120 is 1.02
//    and 6144 1.05 times as fast (in four programs, (1, 16384, 4096), 1.05).
//  * bf16 of up to 20 columns a workgroup not past 320 blocks: (1, 5120,
//    25600), 400 blocks, 51.4 us against 48.4, (1, 5120, 28672) 57.7 against
//    55.7; 20480 level, 16384 1.01 times as fast, and in 24 columns, (1, 6144,
//    28672), 1.05;
//  * up to four rows not with a second row tile of one or two columns: (1,
//    4336, 11264) in 17 23.5 us against 21.4, e4m3 (2, 4352, 2816) 6.9 against
//    6.6, while (1, 5120, 5120) in 20 is level and e4m3 1.07 times as fast.
bool stream_pays(bool bf16, int64_t M, int64_t kbytes, int64_t ldw, int64_t bn,
                 int64_t progs, int64_t groups, int64_t q) {
    int64_t blocks = 11;
    if (bf16 && q * bn <= 20 && kbytes > 320 * 128) return false;
    if (M <= 4 && q * bn > 16 && q * bn <= 18) return false;
    if (M <= 4 && bn <= 16 && q > 1) {
        if (bf16 && q == 2 && q * bn * ldw % (256 * 1024) == 0) return false;
        const int64_t nkb = (kbytes + 127) / 128;
        const int64_t dealt = (nkb + kStreamWaves - 1) / kStreamWaves *
                              kStreamWaves;
        if (bf16 && M <= 2 && 10 * nkb <= 9 * dealt) return false;
        if (bf16)
            blocks = M > 2 ? 16 : ldw % 128 ? 64 : 24;
        else if (M <= 2 && q <= 5)
            blocks = 16;
    }
    return kbytes > blocks * 128 && 20 * progs >= 17 * q * groups;
}

template <int WDT, bool CBF16>
hipError_t launch_stream(const SkinnyArgs &a, int q, int grid, size_t lds,
                         hipStream_t st) {
    static LdsRequest request;
    const hipError_t ready = request(
        {reinterpret_cast<const void *>(&skinny_stream_kernel<WDT, CBF16>)},
        160 * 1024);
    if (ready != hipSuccess) return ready;
    hipLaunchKernelGGL((skinny_stream_kernel<WDT, CBF16>), dim3(grid),
                       dim3(kStreamWaves * 64), lds, st, a, q);
    return hipGetLastError();
}

template <int WDT, int KS, int RT>
hipError_t launch_ks(int c_bf16, const SkinnyArgs &a, hipStream_t st) {
    dim3 grid((a.N + a.bn - 1) / a.bn, a.splitk), block(KS * 64);
    if (c_bf16)
        hipLaunchKernelGGL((gemm_skinny_kernel<WDT, KS, true, RT>), grid,
                           block, 0, st, a);
    else
        hipLaunchKernelGGL((gemm_skinny_kernel<WDT, KS, false, RT>), grid,
                           block, 0, st, a);
    return hipGetLastError();
}

template <int WDT, int RT>
hipError_t launch_w(int c_bf16, int ksplit, const SkinnyArgs &a,
                    hipStream_t st) {
    switch (ksplit) {
    case 1: return launch_ks<WDT, 1, RT>(c_bf16, a, st);
    case 2: return launch_ks<WDT, 2, RT>(c_bf16, a, st);
    case 4: return launch_ks<WDT, 4, RT>(c_bf16, a, st);
    case 8: return launch_ks<WDT, 8, RT>(c_bf16, a, st);
    case 16: return launch_ks<WDT, 16, RT>(c_bf16, a, st);
    default: return hipErrorInvalidValue;
    }
}

template <int WDT>
hipError_t launch_bn(int c_bf16, int bn, int ksplit, const SkinnyArgs &a,
                     hipStream_t st) {
    if (bn != a.bn || bn < 1 || bn > 32) return hipErrorInvalidValue;
    if (bn <= 16) return launch_w<WDT, 1>(c_bf16, ksplit, a, st);
    return launch_w<WDT, 2>(c_bf16, ksplit, a, st);
}

// LDS budget of the staged normalisation weights (one program's K range)
constexpr size_t kNormLdsMax = 32768;

template <int WDT, int RT>
hipError_t launch_norm_rt(int c_bf16, int ksplit, const SkinnyNormArgs &a,
                          hipStream_t st) {
    dim3 grid((a.s.N + a.s.bn - 1) / a.s.bn, a.s.splitk);
    // the fused normalisation runs with four wavefronts per program
    if (ksplit != 4) return hipErrorInvalidValue;
    dim3 block(4 * 64);
    constexpr int KSTEP = WDT == TG_BF16 ? 32 : 64;
    const size_t lds = (size_t)a.s.steps_per_split * KSTEP * 2;
    if (lds <= kNormLdsMax) {
        if (c_bf16)
            hipLaunchKernelGGL((gemm_skinny_norm_kernel<WDT, 4, true, RT, 2>),
                               grid, block, lds, st, a);
        else
            hipLaunchKernelGGL((gemm_skinny_norm_kernel<WDT, 4, false, RT, 2>),
                               grid, block, lds, st, a);
    } else {
        if (c_bf16)
            hipLaunchKernelGGL((gemm_skinny_norm_kernel<WDT, 4, true, RT, 1>),
                               grid, block, 0, st, a);
        else
            hipLaunchKernelGGL((gemm_skinny_norm_kernel<WDT, 4, false, RT, 1>),
                               grid, block, 0, st, a);
    }
    return hipGetLastError();
}

template <int WDT>
hipError_t launch_norm_w(int c_bf16, int bn, int ksplit,
                         const SkinnyNormArgs &a, hipStream_t st) {
    if (bn != a.s.bn || bn < 1 || bn > 32) return hipErrorInvalidValue;
    if (bn <= 16) return launch_norm_rt<WDT, 1>(c_bf16, ksplit, a, st);
    return launch_norm_rt<WDT, 2>(c_bf16, ksplit, a, st);
}

}  // namespace

hipError_t launch_skinny_merge(int c_bf16, const SkinnyArgs &a, bool norm,
                               float eps, hipStream_t st) {
    dim3 grid((a.N + a.bn - 1) / a.bn), block(256);
    if (c_bf16) {
        if (norm)
            hipLaunchKernelGGL((skinny_merge_kernel<true, true>), grid, block,
                               0, st, a, eps);
        else
            hipLaunchKernelGGL((skinny_merge_kernel<true, false>), grid,
                               block, 0, st, a, eps);
    } else {
        if (norm)
            hipLaunchKernelGGL((skinny_merge_kernel<false, true>), grid,
                               block, 0, st, a, eps);
        else
            hipLaunchKernelGGL((skinny_merge_kernel<false, false>), grid,
                               block, 0, st, a, eps);
    }
    return hipGetLastError();
}

hipError_t launch_skinny_norm(int w_dtype, int c_bf16, int bn, int ksplit,
                              const SkinnyNormArgs &a, hipStream_t st) {
    if (w_dtype == TG_BF16)
        return launch_norm_w<TG_BF16>(c_bf16, bn, ksplit, a, st);
    if (w_dtype == TG_FP8_E4M3)
        return launch_norm_w<TG_FP8_E4M3>(c_bf16, bn, ksplit, a, st);
    return hipErrorInvalidValue;
}

int32_t skinny_stream(int w_dtype, int64_t M, int64_t N, int64_t K,
                      int64_t ldx, int64_t ldw, int32_t bn, int cus) {
    const int64_t wes = w_dtype == TG_BF16 ? 2 : 1;
    if (!stream_lds(K * wes, M, K, ldx)) return 0;
    // one workgroup per compute unit
    const int64_t progs = (N + bn - 1) / bn;
    const int64_t groups = cus > 0 ? cus : 256;
    const int64_t q = (progs + groups - 1) / groups;
    const int64_t span = (q * bn + 16) * ldw * wes;
    return span < 0x7fffffff && stream_pays(wes == 2, M, K * wes, ldw * wes,
                                            bn, progs, groups, q)
               ? (int32_t)q : 0;
}

hipError_t launch_skinny(int w_dtype, int c_bf16, int bn, int ksplit,
                         const SkinnyArgs &a, int stream, hipStream_t st) {
    if (stream > 0) {
        const int64_t progs = (a.N + (int64_t)bn - 1) / bn;
        const int grid = (int)((progs + stream - 1) / stream);
        const size_t lds = (size_t)stream_lds(
            w_dtype == TG_BF16 ? a.K * (int64_t)2 : a.K, a.M, a.K, a.ldx);
        if (w_dtype == TG_BF16)
            return c_bf16
                       ? launch_stream<TG_BF16, true>(a, stream, grid, lds, st)
                       : launch_stream<TG_BF16, false>(a, stream, grid, lds,
                                                       st);
        return c_bf16
                   ? launch_stream<TG_FP8_E4M3, true>(a, stream, grid, lds, st)
                   : launch_stream<TG_FP8_E4M3, false>(a, stream, grid, lds,
                                                       st);
    }
    if (w_dtype == TG_BF16)
        return launch_bn<TG_BF16>(c_bf16, bn, ksplit, a, st);
    if (w_dtype == TG_FP8_E4M3)
        return launch_bn<TG_FP8_E4M3>(c_bf16, bn, ksplit, a, st);
    return hipErrorInvalidValue;
}

}  // namespace tg
