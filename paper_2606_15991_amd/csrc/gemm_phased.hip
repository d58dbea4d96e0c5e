// gemm_phased.hip -- the phased schedule of the tiled product: 256 x 256
// sub-tensors, 128-byte K tiles (64 bf16, 128 e4m3), eight wavefronts of
// 128 x 64 outputs in two groups of four, one of each group on every SIMD.
//
// A K tile is contracted in four phases, one quarter (64 x 32 outputs) of
// the wavefront's block each.  A phase has two slots, with a workgroup
// barrier after each: in the memory slot the wavefront reads the fragments
// that the phase needs from LDS and issues one sixteenth of a tile two tiles
// ahead; in the compute slot it issues 16 (e4m3: 8) matrix instructions.
// The second group runs one slot behind the first, so that on every SIMD one
// wavefront contracts while the other reads.  Half tiles (64 of each
// wavefront's 128 A rows, 32 of its 64 B columns) are the unit of LDS reuse:
// the loads of a half are issued as soon as both groups have read it, five
// to six phases before their data are needed, against one tile period or
// less where whole stages change hands.
//
// What bounds it.  Random operands: power.  The matrix cores, LDS reads and
// direct loads of this loop pull the clock to about 1.9 GHz; with operands
// of zeros the same launch takes 610 us at 8192^3 (1800 TFLOP/s).  Hence the
// 16x16x32 (e4m3: 16x16x128) instruction, which sums twice the K per
// accumulator update of the 32x32x16 one: matrix instructions alone on
// random operands run at 2095 TFLOP/s against 1828, with this loop's LDS
// reads and loads 1530 against 1380, this kernel 763 us against 798.  In
// cycles, the direct loads: a slot takes 340 to 350 cycles against 256 of
// matrix work (by the counters the matrix cores are busy 76 % of a compute
// unit's cycles), 285 without them (the load path moves 64 bytes a clock and
// a wavefront waits while it is busy).  LDS: bf16 2 % of its cycles are bank
// conflicts, e4m3 49 %, whose lanes read two neighbouring chunks of a row, and
// transposing reads of a k-major B 26 %; e4m3 is busy 74 % all the same.  Issuing the loads between matrix
// instructions (832 us), before the reads, staggered over the wavefronts
// (+-1 %), or with one barrier per two phases (757 us, but e4m3 5 % slower)
// is no better.
//
// Measured against the schedules it replaces as defaults (same box each):
// bf16 8192^3 B stored N x K 756 us against 864 (cross-tile ring), K x N 791
// against 865 (lock-step), e4m3 8192^3 389 against 456 (lock-step), 4096^2 x
// 32768 747 against 927 (cross-tile ring with an L2 warm-up), bf16x6 4096^3
// 679 against 782, 64 mixed problems in one grouped launch 2108 against 2431.
#include <type_traits>

#include "tg_tiled.hpp"

namespace tg {
namespace {

typedef __attribute__((address_space(3))) i32x4 lds_i32x4;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;

// NF fragments of 16 rows by one K tile (128 bytes): bf16 two K steps of
// 32, e4m3 one of 128.
template <class C, int NF>
struct PhFrag {
    static constexpr bool F8 = C::DTYPE == TG_FP8_E4M3;
    static constexpr int NQ = F8 ? 1 : 2;
    typedef std::conditional_t<F8, i32x8, i32x4> V;
    V v[NF][NQ];
};

template <int S>
using Int = std::integral_constant<int, S>;

// acc += (b . a)^T: the B fragment is the instruction's first operand, so
// that a lane holds four consecutive columns of one output row.  In assembly
// with the accumulator in accumulation registers throughout, since the
// compiler gives each copy of the K loop's instructions its own accumulator
// registers and moves (and spills) 128 registers between them.  Consecutive
// instructions on one accumulator need no wait states; a reader of the
// results must call mfma_drain() first.
template <class C>
__device__ __forceinline__ void ph_mfma(
    const typename PhFrag<C, 1>::V &a, const typename PhFrag<C, 1>::V &b,
    f32x4 &acc) {
#ifdef __HIP_DEVICE_COMPILE__   // (no such registers in the host pass)
    if constexpr (C::DTYPE == TG_FP8_E4M3)
        asm volatile("v_mfma_f32_16x16x128_f8f6f4 %0, %1, %2, %0"
                     : "+a"(acc) : "v"(b), "v"(a));
    else
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"
                     : "+a"(acc) : "v"(b), "v"(a));
#endif
}

// acc = 0 (a product of zeros, so that the accumulator is born in its
// accumulation registers).
__device__ __forceinline__ void mfma_zero(f32x4 &acc) {
#ifdef __HIP_DEVICE_COMPILE__
    const i32x4 z = {0, 0, 0, 0};
    asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %1, 0"
                 : "=a"(acc) : "v"(z));
#endif
}

__device__ __forceinline__ void mfma_drain() {
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
}

// At most N LDS accesses of this wavefront in flight (vmcnt and expcnt at
// their no-wait maxima).
template <int N>
__device__ __forceinline__ void wait_lds_le() {
    static_assert(N >= 0 && N < 16, "lgkmcnt range");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4) | (N << 8));
}

__device__ __forceinline__ void slot_end() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// Two 16-byte-per-lane loads, at byte offsets v0 and v1 (+ soff), into LDS
// at base + OFF and base + OFF + 8192 (+ 16 * lane).  One block, so that
// nothing comes between: the wait states cover scalar registers that a
// vector instruction just wrote (five) and M0 (one).
template <int OFF>
__device__ __forceinline__ void ph_dma2(const i32x4 &srd, uint32_t base,
                                        const uint32_t (&v)[2], int soff) {
    asm volatile(
        "s_add_u32 m0, %0, %5\n\ts_nop 3\n\t"
        "buffer_load_dwordx4 %1, %3, %4 offen lds\n\t"
        "s_add_u32 m0, %0, %6\n\ts_nop 0\n\t"
        "buffer_load_dwordx4 %2, %3, %4 offen lds"
        :
        : "s"(base), "v"(v[0]), "v"(v[1]), "s"(srd),
          "s"(__builtin_amdgcn_readfirstlane(soff)), "i"(OFF),
          "i"(OFF + 8192)
        : "memory", "m0", "scc");
}

// One such load.
template <int OFF>
__device__ __forceinline__ void ph_dma1(const i32x4 &srd, uint32_t base,
                                        uint32_t v, int soff) {
    asm volatile(
        "s_add_u32 m0, %0, %4\n\ts_nop 3\n\t"
        "buffer_load_dwordx4 %1, %2, %3 offen lds"
        :
        : "s"(base), "v"(v), "s"(srd),
          "s"(__builtin_amdgcn_readfirstlane(soff)), "i"(OFF)
        : "memory", "m0", "scc");
}

__device__ __forceinline__ int ph_swz(int row) { return (row >> 1) & 7; }

// Wavefronts of TM x 64 outputs, as 16 x 16 blocks.
template <class C>
struct PhStore {
    static_assert(C::TN == 64, "four column blocks a wavefront");
    static constexpr int NRB = C::TM / 16;
    typedef f32x4 Acc[NRB][4];

    // Store the accumulators into the owned sub-tensor.  Result layout of
    // the transposed 16 x 16 product: lane l, register v holds row l % 16,
    // column 4 (l / 16) + v.  Stores coalesce over consecutive lanes only, so
    // each wavefront passes blocks of 16 rows by 128 bytes (binary32 32
    // columns, bf16 64) through 2 KiB of LDS of its own and stores eight
    // rows of eight lanes by 16 bytes (256 KiB of one sub-tensor alone on
    // the chip: 8300 cycles in the registers' order, 5600 in this one).
    // A lane's 16 bytes that straddle N go out element by element; rows past
    // M and columns past N get an out-of-range offset, which the hardware
    // drops.  The accumulators are read by ordered assembly: left to itself
    // the compiler copies all 128 at once and spills.
    template <bool SCALED>
    __device__ __forceinline__ static void store(const Job &j, Acc &acc,
                                                 const char *scl, char *smem,
                                                 int lane, int wave) {
        const int wm = wave / C::WN, wn = wave % C::WN;
        constexpr int OES = C::CBF16 ? 2 : 4, VW = 16 / OES;
        int lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)j.ldc);
        int hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)(j.ldc >> 32));
        // (formed here, not held across the K loop)
        asm volatile("" : "+s"(lo), "+s"(hi));
        const int64_t ldc =
            (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
        char *base = static_cast<char *>(j.c) +
                     ((int64_t)j.m0 * ldc + j.n0) * OES;
        const __amdgpu_buffer_rsrc_t r = make_rsrc(
            base, sat_bytes(((int64_t)(j.M - j.m0 - 1) * ldc +
                             (j.N - j.n0)) * OES));
        // this lane's place in a stored block: rows sr and sr + 8, bytes
        // 16 sc
        const int sr = lane >> 3, sc = lane & 7;
        const int r0 = wm * C::TM + sr, c0 = wn * 64 + sc * VW;
        const int rows_left = j.M - j.m0 - r0, cols_left = j.N - j.n0 - c0;
        // and in a block of results: row ar, 16-byte chunks ag and ag + 4
        const int ar = lane & 15, ag = lane >> 4;
        const uint32_t blk = lds_addr(smem) + C::NS * C::STAGE +
                             C::NSLOT * C::SCALE_SLOT + wave * 2048;
        const uint32_t w0 = blk + ar * 128 + ((ag ^ ph_swz(ar)) << 4);
        const uint32_t w1 = blk + ar * 128 + (((ag + 4) ^ ph_swz(ar)) << 4);
        const uint32_t s0 = blk + sr * 128 + ((sc ^ ph_swz(sr)) << 4);
        const uint32_t s1 = blk + (sr + 8) * 128 + ((sc ^ ph_swz(sr + 8)) << 4);
        // bf16 rows that start inside a dword
        const bool split = C::CBF16 &&
                           (((reinterpret_cast<uintptr_t>(base) >> 1) |
                             (uintptr_t)ldc) & 1);
        // whole sub-tensors: no per-store tests
        const bool inner = j.n0 + C::BN <= j.N && j.m0 + C::BM <= j.M &&
                           !split;
        const bool ragged = j.n0 + C::BN > j.N && j.N % VW != 0;
        const float *lsa = reinterpret_cast<const float *>(scl);
        const float *lsb = lsa + C::BM;
        float sb[SCALED ? 16 : 1];
        if constexpr (SCALED) {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                // column of register e % 4 of fragment e / 4
                const int c = wn * 64 +
                              (C::CBF16 ? (e >> 3) * 32 + 8 * ag + (e & 7)
                                        : (e >> 2) * 16 + 4 * ag + (e & 3));
                sb[e] = j.scale_b ? lsb[c] : 1.f;
            }
        }
        const uint32_t off0 = (uint32_t)((r0 * ldc + c0) * OES);
#pragma unroll
        for (int i = 0; i < NRB; ++i) {
            float sa = 1.f;
            if constexpr (SCALED)
                if (j.scale_a) sa = lsa[wm * C::TM + i * 16 + ar];
#pragma unroll
            for (int h = 0; h < 8 / VW; ++h) {   // 2, bf16 1
                // VW / 2 fragments of this block: two chunks a lane
                float x[2 * VW];
#pragma unroll
                for (int v = 0; v < 2 * VW; ++v) {
                    const int e = h * 2 * VW + v;
                    const float a = acc[i][e >> 2][e & 3];
#ifdef __HIP_DEVICE_COMPILE__
                    asm volatile("v_accvgpr_read_b32 %0, %1"
                                 : "=v"(x[v]) : "a"(a));
#endif
                    if constexpr (SCALED) x[v] = x[v] * sb[e] * sa;
                }
                u32x4 wa, wb;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if constexpr (C::CBF16) {
                        wa[q] = f32x2_to_bf16x2(x[2 * q], x[2 * q + 1]);
                        wb[q] = f32x2_to_bf16x2(x[VW + 2 * q],
                                                x[VW + 2 * q + 1]);
                    } else {
                        wa[q] = as_u32(x[q]);
                        wb[q] = as_u32(x[VW + q]);
                    }
                }
                // (a wavefront's LDS accesses execute in order)
                *reinterpret_cast<lds_u32x4 *>(w0) = wa;
                *reinterpret_cast<lds_u32x4 *>(w1) = wb;
                __builtin_amdgcn_wave_barrier();
                const u32x4 ya = *reinterpret_cast<const lds_u32x4 *>(s0);
                const u32x4 yb = *reinterpret_cast<const lds_u32x4 *>(s1);
                __builtin_amdgcn_wave_barrier();
                const uint32_t off = off0 + (uint32_t)(i * 16 * ldc * OES) +
                                     h * 128;
                const uint32_t off8 = off + (uint32_t)(8 * ldc * OES);
                if (inner) {
                    __builtin_amdgcn_raw_buffer_store_b128(ya, r, off, 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b128(yb, r, off8, 0, 0);
                } else {
                    const int cl = cols_left - h * 32;
                    put_edge<VW>(r, base, ya, off, i * 16 < rows_left, cl,
                                 split, ragged);
                    put_edge<VW>(r, base, yb, off8, i * 16 + 8 < rows_left,
                                 cl, split, ragged);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (j.wcount) {
            // instrumented launches: one count per stored element
#pragma unroll 1
            for (int i = 0; i < 2 * NRB; ++i) {
                if (i * 8 >= rows_left) continue;
#pragma unroll 1
                for (int e = 0; e < 8; ++e) {
                    const int c = (e / VW) * 32 + e % VW;
                    if (c < cols_left)
                        atomicAdd(&j.wcount[(int64_t)(j.m0 + r0 + i * 8) *
                                                j.N + j.n0 + c0 + c], 1);
                }
            }
        }
    }
    // 16 bytes at an edge of the output: cl columns of it are left.
    template <int VW>
    __device__ __forceinline__ static void put_edge(
        const __amdgpu_buffer_rsrc_t &r, char *base, const u32x4 &w,
        uint32_t off, bool row_in, int cl, bool split, bool ragged) {
        const bool in = row_in && cl >= VW;
        if (!split)
            __builtin_amdgcn_raw_buffer_store_b128(
                w, r, in ? off : kOutOfRange, 0, 0);
        else if (in)
            __builtin_memcpy(base + off, &w, 16);
        if (ragged) {
#pragma unroll
            for (int v = 0; v < VW - 1; ++v) {
                const uint32_t o = row_in && !in && v < cl
                                       ? off + v * (16 / VW) : kOutOfRange;
                if constexpr (VW == 8)
                    __builtin_amdgcn_raw_buffer_store_b16(
                        (unsigned short)(w[v >> 1] >> (16 * (v & 1))), r, o,
                        0, 0);
                else
                    __builtin_amdgcn_raw_buffer_store_b32(w[v & 3], r, o, 0,
                                                          0);
            }
        }
    }
};

// PL: the operands are planes of a split binary32 product, side by side
// along K (K % 64 == 0 elements each), and the K loop runs over products of
// planes: block b of kp elements multiplies plane a of A and plane b of B as
// GemmArgs says.  A plane that several products read is stored once.
template <class C, bool PL = false>
struct Phased {
    static_assert(C::BM == 256 && C::BN == 256 && C::RBY == 128 &&
                      C::NW == 8 && C::WM == 2 && C::FM == 4 && C::FN == 2,
                  "256 x 256 tiles, 2 x 4 wavefronts of 128 x 64");
    static constexpr int HALF = 128 * 128;       // bytes per half region
    // two stages, the scale slots and a 2 KiB store block per wavefront
    static constexpr int SMEM =
        2 * C::STAGE + C::NSLOT * C::SCALE_SLOT + 8 * 2048;
    static_assert(SMEM <= 163840, "160 KiB of LDS");
    using FA = PhFrag<C, 4>;      // half of A's rows of a wavefront
    using FB = PhFrag<C, 2>;      // half of B's columns
    static constexpr int NQ = FA::NQ;
    typedef PhStore<C> Store;
    typedef typename Store::Acc Acc;

    // LDS stage: A half 0, A half 1, B half 0, B half 1, each 128 rows of
    // 128 bytes with 16-byte chunk c of row r at c ^ ((r >> 1) & 7) (k-major
    // B: 64 rows of k by 128 columns), 16 blocks of 1 KiB, block i loaded by
    // wavefront i % 8.
    char *smem;
    int tid, lane, wave, wm, wn;
    uint32_t aoff[2][2], boff[2][4];   // LDS addresses, by stage
    uint32_t lbase;   // LDS address of this wavefront's 1 KiB block 0

    Job j;
    i32x4 sa, sb;
    uint32_t va[2][2], vb[2][2];
    int nk, head;     // K tiles; 1 when tile 0 of the sequence is K's tail
    // PL: byte offsets along K of the product tile that is loaded next (and
    // of A's tile before it), bytes of a plane, K tiles left of the current
    // product and the products still to come
    int soa1, soa, sob, kpb, left_pl;
    uint32_t ord_a, ord_b;

    // The K tiles of a sub-tensor in the order they are contracted: a
    // partial last tile comes first, so that all later loads are whole.
    __device__ __forceinline__ int k0_of(int q) const {
        return (head ? (q == 0 ? nk - 1 : q - 1) : q) * C::BK;
    }
    // row of the tile in row lr of half h
    __device__ __forceinline__ static int a_row(int lr, int h) {
        return (lr >> 6) * 128 + h * 64 + (lr & 63);
    }
    // (bf16 output: B rows are placed so that the two fragments of a half
    // give a lane eight consecutive columns, 16 bytes of a row)
    __device__ __forceinline__ static int b_row(int lr, int h) {
        const int p = lr & 31;
        const int n = C::CBF16 ? 8 * ((p >> 2) & 3) + 4 * (p >> 4) + (p & 3)
                               : p;
        return (lr >> 5) * 64 + h * 32 + n;
    }
    __device__ __forceinline__ static int swz7(int lr) { return ph_swz(lr); }

    __device__ __forceinline__ void init(char *s) {
        smem = s;
        tid = threadIdx.x;
        lane = tid & 63;
        wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        lbase = lds_addr(s) + wave * 1024;
        wm = wave >> 2;
        wn = wave & 3;
        const int r = lane & 15, grp = lane >> 4;
        const uint32_t base = lds_addr(s);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int ch = C::DTYPE == TG_FP8_E4M3 ? 2 * grp + q
                                                   : 4 * q + grp;
            const int c = (ch ^ swz7(r)) << 4;
            aoff[0][q] = base + (wm * 64 + r) * 128 + c;
            boff[0][q] = base + 2 * HALF + (wn * 32 + r) * 128 + c;
            aoff[1][q] = aoff[0][q] + C::STAGE;
            // (held: not re-derived in the K loop)
            asm volatile("" : "+v"(aoff[1][q]));
        }
        if constexpr (C::B_KMAJOR) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                // fragment q / 2, rows 4 (q % 2) .. + 3 of the lane group's
                // eight; see read_b
                const int n = wn * 32 +
                              (C::CBF16 ? 4 * (q >> 1) + 8 * (r & 3)
                                        : 16 * (q >> 1) + 4 * (r & 3));
                const int k = grp * 8 + (q & 1) * 4 + (r >> 2);
                boff[0][q] = base + 2 * HALF + k * 256 +
                             (((n >> 3) ^ kswz(k)) << 4) + ((n & 7) << 1);
            }
        }
#pragma unroll
        for (int q = 0; q < (C::B_KMAJOR ? 4 : 2); ++q) {
            boff[1][q] = boff[0][q] + C::STAGE;
            asm volatile("" : "+v"(boff[1][q]));
        }
    }
    __device__ __forceinline__ static int kswz(int k) {
        constexpr uint32_t tab = 0u | (4u << 8) | (10u << 16) | (14u << 24);
        return (tab >> (8 * (k & 3))) & 0xff;
    }

    __device__ __forceinline__ void set_job(const Job &nj) {
        j = nj;
        // (uniform, also where the problem comes from a table in memory)
        j.K = __builtin_amdgcn_readfirstlane(j.K);
        nk = (j.K + C::BK - 1) / C::BK;
        head = j.K % C::BK ? 1 : 0;
        sa = make_srd(j.a_row, sat_bytes(j.a_rem));
        if constexpr (!C::B_KMAJOR) sb = make_srd(j.b_row, sat_bytes(j.b_rem));
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int lr = (i * 8 + wave) * 8 + (lane >> 3);
            const int kc = (lane & 7) ^ swz7(lr);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                va[h][i] = (uint32_t)((a_row(lr, h) * j.lda + kc * C::EPC) *
                                      C::ES);
                if constexpr (!C::B_KMAJOR) {
                    vb[h][i] = (uint32_t)(
                        (b_row(lr, h) * j.ldb + kc * C::EPC) * C::ES);
                } else {
                    const int k = (i * 8 + wave) * 4 + (lane >> 4);
                    const int lc = (lane & 15) ^ kswz(k);
                    const int col = (lc >> 2) * 64 + h * 32 + (lc & 3) * 8;
                    vb[h][i] = j.n0 + col < j.N
                                   ? (uint32_t)((k * j.ldb + col) * C::ES)
                                   : kOutOfRange;
                }
            }
        }
    }
    // Byte offset of sequence tile q >= 1 along K (K tiles are 128 bytes).
    __device__ __forceinline__ int soff(int q) const {
        return (q - head) << 7;
    }
    // PL: offsets of the first product's first tile, and on to the next.
    __device__ __forceinline__ void next_product() {
        soa = (int)(ord_a & 0xf) * kpb;
        sob = (int)(ord_b & 0xf) * kpb;
        ord_a >>= 4;
        ord_b >>= 4;
        left_pl = kpb >> 7;
    }
    __device__ __forceinline__ void next_offsets() {
        soa1 = soa;
        soa += 128;
        sob += 128;
        if (--left_pl == 0) next_product();
    }
    // Half H of A / B into stage S, K offset so (row mode; k-major: srd is
    // the tile's own descriptor).
    template <int S, int H>
    __device__ __forceinline__ void issue_a(int so) const {
        ph_dma2<S * C::STAGE + H * HALF>(sa, lbase, va[H], so);
    }
    template <int S, int H>
    __device__ __forceinline__ void issue_b(int so) const {
        ph_dma2<S * C::STAGE + (2 + H) * HALF>(sb, lbase, vb[H], so);
    }
    // Descriptor of a k-major B from offset so along K, not tile 0's: all its rows lie
    // inside K, columns past N are masked by their offsets.
    __device__ __forceinline__ void kmajor_tile(int so) {
        if constexpr (C::B_KMAJOR)
            sb = make_srd(j.b_row + (int64_t)(so / C::ES) * j.ldb * C::ES,
                          0x7fffffffu);
    }
    __device__ __forceinline__ int bsoff(int so) const {
        return C::B_KMAJOR ? 0 : so;
    }
    // tile 0 of the sequence, possibly K's tail: chunks not wholly inside K
    // load as zeros
    __device__ __forceinline__ void issue_tile0() {
        const int k0 = PL ? 0 : k0_of(0);
        const int oa = PL ? soa : k0 * C::ES, ob = PL ? sob : k0 * C::ES;
        constexpr bool KM = C::B_KMAJOR;
        i32x4 b0 = sb;
        if constexpr (KM) {
            const int64_t skip = (int64_t)(ob / C::ES) * j.ldb * C::ES;
            b0 = make_srd(j.b_row + skip, sat_bytes(j.b_rem - skip));
        }
        auto put = [&](auto D, const i32x4 &srd, const uint32_t (&v)[2],
                       bool rows_of_k, int so) {
            uint32_t w[2] = {v[0], v[1]};
            if (!rows_of_k) {
                if (!chunk_in(0, k0)) w[0] = kOutOfRange;
                if (!chunk_in(1, k0)) w[1] = kOutOfRange;
            }
            ph_dma2<D.value>(srd, lbase, w, rows_of_k ? 0 : so);
        };
        put(Int<2 * HALF>{}, b0, vb[0], KM, ob);
        put(Int<0>{}, sa, va[0], false, oa);
        put(Int<3 * HALF>{}, b0, vb[1], KM, ob);
        put(Int<HALF>{}, sa, va[1], false, oa);
    }
    __device__ __forceinline__ bool chunk_in(int i, int k0) const {
        const int lr = (i * 8 + wave) * 8 + (lane >> 3);
        const int kc = (lane & 7) ^ swz7(lr);
        return k0 + (kc + 1) * C::EPC <= j.K;
    }
    // the first tiles of a sub-tensor: tile 0 and all of tile 1 but its A
    // half 1
    __device__ __forceinline__ void issue_first() {
        if (nk > 0) issue_tile0();
        if constexpr (PL) next_offsets();
        if (nk > 1) {
            const int oa = PL ? soa : soff(1), ob = PL ? sob : soff(1);
            kmajor_tile(ob);
            issue_b<1, 0>(bsoff(ob));
            issue_a<1, 0>(oa);
            issue_b<1, 1>(bsoff(ob));
        }
        if constexpr (PL) next_offsets();
    }
    // The chunk that straddles K was loaded as zeros: its K % EPC valid
    // elements of every row, one by one.
    __device__ __forceinline__ void fill_tail() {
        const int rem = j.K % C::EPC, kbase = j.K - rem;
        const int chunk = (kbase - k0_of(0)) / C::EPC;
        auto put = [&](char *dst, const char *src, bool ok) {
            for (int e = 0; e < rem; ++e) {
                if constexpr (C::ES == 2)
                    reinterpret_cast<uint16_t *>(dst)[e] =
                        ok ? reinterpret_cast<const uint16_t *>(src)[e] : 0;
                else
                    reinterpret_cast<uint8_t *>(dst)[e] =
                        ok ? reinterpret_cast<const uint8_t *>(src)[e] : 0;
            }
        };
        for (int e = tid; e < 256; e += C::THREADS) {
            const int h = e >> 7, lr = e & 127, row = a_row(lr, h);
            put(smem + h * HALF + lr * 128 + ((chunk ^ swz7(lr)) << 4),
                j.a + ((int64_t)(j.m0 + row) * j.lda + kbase) * C::ES,
                j.m0 + row < j.M);
        }
        if constexpr (!C::B_KMAJOR) {
            for (int e = tid; e < 256; e += C::THREADS) {
                const int h = e >> 7, lr = e & 127, row = b_row(lr, h);
                put(smem + (2 + h) * HALF + lr * 128 +
                        ((chunk ^ swz7(lr)) << 4),
                    j.b + ((int64_t)(j.n0 + row) * j.ldb + kbase) * C::ES,
                    j.n0 + row < j.N);
            }
        }
    }
    __device__ __forceinline__ static i32x4 ld(uint32_t p) {
        return *reinterpret_cast<const lds_i32x4 *>(p);
    }
    template <int NF>
    __device__ __forceinline__ static void read_rows(PhFrag<C, NF> &o,
                                                     const uint32_t *p,
                                                     uint32_t d) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const uint32_t e = d + f * 16 * 128;
            if constexpr (FA::F8) {
                const i32x4 lo = ld(p[0] + e), hi = ld(p[1] + e);
                o.v[f][0] = i32x8{lo[0], lo[1], lo[2], lo[3],
                                  hi[0], hi[1], hi[2], hi[3]};
            } else {
                o.v[f][0] = ld(p[0] + e);
                o.v[f][1] = ld(p[1] + e);
            }
        }
    }
    template <int S>
    __device__ __forceinline__ void read_a(FA &a, int h) const {
        read_rows(a, aoff[S], h * HALF);
    }
    // k-major: two transposing reads per fragment and K step.  In each
    // 16-lane group lane r names row k = kb + r / 4 at columns c0 +
    // 4 (r % 4) .. + 3 and lane i receives column c0 + i at rows kb ..
    // kb + 3.
    template <int S>
    __device__ __forceinline__ void read_b(FB &b, int h) const {
        if constexpr (C::B_KMAJOR) {
#pragma unroll
            for (int f = 0; f < 2; ++f)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    i32x4 out;
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const s16x4 v =
                            __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                (lds_s16x4 *)(boff[S][2 * f + u] + h * HALF +
                                              q * 32 * 256));
                        const uint32_t v0 = (uint16_t)v[0];
                        const uint32_t v1 = (uint16_t)v[1];
                        const uint32_t v2 = (uint16_t)v[2];
                        const uint32_t v3 = (uint16_t)v[3];
                        out[2 * u] = (int)(v0 | (v1 << 16));
                        out[2 * u + 1] = (int)(v2 | (v3 << 16));
                    }
                    b.v[f][q] = out;
                }
        } else {
            read_rows(b, boff[S], h * HALF);
        }
    }
    template <int HA, int HB>
    __device__ __forceinline__ static void quad(const FA &a, const FB &b,
                                                Acc &acc) {
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    ph_mfma<C>(a.v[i][q], b.v[j][q],
                               acc[4 * HA + i][2 * HB + j]);
    }
    // barrier, contract, barrier
    template <int HA, int HB>
    __device__ __forceinline__ static void slots(const FA &a, const FB &b,
                                                 Acc &acc) {
        slot_end();
        __builtin_amdgcn_s_setprio(1);
        quad<HA, HB>(a, b, acc);
        __builtin_amdgcn_s_setprio(0);
        slot_end();
    }
    // Wait until the half that the next phase reads has landed.  Halves are
    // loaded in the order of their first reads, two loads of a wavefront
    // each, and five of them are issued between a half's own issue and this
    // wait; fewer (W1, W0) in the last tile but one and in the last, whose
    // later halves do not exist.
    template <int W1, int W0>
    __device__ __forceinline__ static void wait_loads(int left) {
        wait_vmem_le<10>();
        if (__builtin_expect(left <= 2, 0)) {
            if (left == 2) wait_vmem_le<W1>();
            else wait_vmem_le<W0>();
        }
    }
    // K tile of the sequence in stage S, `left` tiles to go with it; x holds
    // its B half 0, and at the end y holds the next tile's.  so_a1, so_a and
    // so_b: offsets along K of A's next tile and of both operands' tile two
    // further on.
    //
    // Reuse, counted in slots: A half 0, B half 1 and A half 1 are read in the
    // memory slots of phases 1, 2 and 3 and contracted in the slot after, so
    // the second group, one slot behind, has their data two slots after the
    // first group read them; they are loaded over in the first group's
    // memory slots of phases 3, 4 and 1 of the next tile, four slots after.
    // B half 0 is read in phase 4 but contracted only in phase 1 of the next
    // tile, four slots on for the second group, which would be the very slot
    // in which the first group loads over it (phase 2): hence the wait for
    // it at the end of phase 1's memory slot, with phase 1's own eight reads
    // still in flight (a wavefront's LDS reads return in order).
    template <int S>
    __device__ __forceinline__ void tile(FA &a, FB &x, FB &y, Acc &acc,
                                         int left, int so_a1, int so_a,
                                         int so_b) {
        read_a<S>(a, 0);
        if (__builtin_expect(left > 1, 1)) issue_a<1 - S, 1>(so_a1);
        wait_loads<10, 2>(left);
        wait_lds_le<8>();
        slots<0, 0>(a, x, acc);
        read_b<S>(y, 1);
        if (__builtin_expect(left > 2, 1)) {
            kmajor_tile(so_b);
            issue_b<S, 0>(bsoff(so_b));
        }
        wait_loads<8, 0>(left);
        slots<0, 1>(a, y, acc);
        read_a<S>(a, 1);
        if (__builtin_expect(left > 2, 1)) issue_a<S, 0>(so_a);
        wait_loads<6, 0>(left);
        slots<1, 1>(a, y, acc);
        read_b<1 - S>(y, 0);
        if (__builtin_expect(left > 2, 1)) issue_b<S, 1>(bsoff(so_b));
        if constexpr (PL) next_offsets();
        wait_loads<4, 0>(left);
        slots<1, 0>(a, x, acc);
    }

    template <class P>
    __device__ __forceinline__ void start_offsets(const P &prov) {
        if constexpr (PL) {
            ord_a = prov.g.planes_a;
            ord_b = prov.g.planes_b;
            kpb = prov.g.kp * C::ES;
            next_product();
        }
    }
    template <class P>
    __device__ __forceinline__ void run(const P &prov, char *s) {
        const int G = prov.n_prog(), total = prov.count();
        int t = program_slot(blockIdx.x, G);
        if (t >= total) return;
        init(s);
        int njob = 0;
        Acc acc;
        FA a;
        FB x, y;
        set_job(prov.job(t));
        start_offsets(prov);
        tg::issue_scales<C>(j, scale_slot<C>(smem, 0), wave, lane);
        issue_first();
        while (true) {
#pragma unroll
            for (int i = 0; i < 32; ++i) mfma_zero(acc[i >> 2][i & 3]);
            const bool ragged = j.K % C::EPC != 0;
            wait_vmem();      // also the previous sub-tensor's stores
            slot_end();
            if (ragged) {
                fill_tail();
                __syncthreads();
            }
            if (nk > 0) {
                read_b<0>(x, 0);
                if (wm) slot_end();       // one slot behind
                int so = soff(2);
                for (int left = nk;; left -= 2, so += 256) {
                    tile<0>(a, x, y, acc, left, PL ? soa1 : so - 128,
                            PL ? soa : so, PL ? sob : so);
                    if (left == 1) break;
                    tile<1>(a, y, x, acc, left - 1, PL ? soa1 : so,
                            PL ? soa : so + 128, PL ? sob : so + 128);
                    if (left == 2) break;
                }
                if (!wm) slot_end();      // level again: LDS is free
            }
            mfma_drain();
            t += G;
            const bool more = t < total;
            const Job done = j;
            if (more) {
                set_job(prov.job(t));
                start_offsets(prov);
                tg::issue_scales<C>(j, scale_slot<C>(smem, njob + 1), wave,
                                    lane);
                issue_first();
            }
            if (done.scale_a || done.scale_b)
                Store::template store<true>(done, acc,
                                            scale_slot<C>(smem, njob), smem,
                                            lane, wave);
            else
                Store::template store<false>(done, acc, nullptr, smem, lane,
                                             wave);
            if (!more) break;
            ++njob;
        }
    }
};

template <class C, bool PL>
__global__ __launch_bounds__(512)
__attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_phased_kernel(
    GemmArgs g) {
    extern __shared__ __align__(1024) char smem[];
    SingleProvider<C> p{g};
    Phased<C, PL> k;
    k.run(p, smem);
}

template <class C>
__global__ __launch_bounds__(512)
__attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_phased_grouped_kernel(
    const GroupProblem *__restrict__ tab, int n, int total, int G) {
    extern __shared__ __align__(1024) char smem[];
    GroupProvider<C> p{tab, n, total, G};
    Phased<C> k;
    k.run(p, smem);
}

// 128 x 128 sub-tensors: the same two groups of wavefronts one slot apart
// (wavefronts 4 - 7, rows 64 .. 127, behind), but a wavefront's 32 x 64
// outputs take only 48 registers of fragments for a whole K tile, so there
// is one memory slot and one compute slot of 16 instructions per K tile, and
// LDS holds four stages of which three are loaded ahead.  Bound by the memory
// slot, 12 fragment reads and A's two loads of a wavefront; B's two loads in
// front of the compute slot's instructions even the slots out (512 x 5120 x
// 5120 37.6 us, all four in the memory slot 44.9).  Against eight wavefronts
// in step with the same ring: 512 x 5120 x 5120 52.8 us, 2048^3 21.0 against
// 25.3, e4m3 13.4 against 15.5.  Not for a k-major B, whose 16 transposing
// reads make the memory slot longer (52 us against 50).
//
// MIX: bf16 A with e4m3 weights stored N x K (rows of 64 bytes in LDS, chunk
// c of row r at c ^ ((r >> 2) & 3)), decoded to bf16 in the memory slot.  A
// lane then holds 16 consecutive k of a weight row, eight for each K step,
// and reads A's fragments at the same k.
template <class C, bool MIX = false>
struct Phased128 {
    static_assert(C::BM == 128 && C::BN == 128 && C::RBY == 128 &&
                      C::NW == 8 && C::WM == 4 && C::WN == 2 && C::NS == 4,
                  "128 x 128 tiles, 4 x 2 wavefronts of 32 x 64");
    static_assert(!C::B_KMAJOR && (!MIX || C::DTYPE == TG_BF16),
                  "B stored N x K; bf16 by e4m3");
    static constexpr int ABYTES = 128 * 128;
    static constexpr int BROW = MIX ? 64 : 128;
    static constexpr int STG = ABYTES + 128 * BROW;
    static constexpr int LOADS = MIX ? 3 : 4;         // of a wavefront
    static constexpr int SMEM =
        C::NS * C::STAGE + C::NSLOT * C::SCALE_SLOT + 8 * 2048;
    static_assert(SMEM <= 163840, "160 KiB of LDS");
    static constexpr int BES = MIX ? 1 : C::ES;       // bytes of B's elements
    using FA = PhFrag<C, 2>;
    using FB = PhFrag<C, 4>;
    static constexpr int NQ = FA::NQ;
    typedef PhStore<C> Store;
    typedef typename Store::Acc Acc;

    char *smem;
    int tid, lane, wave, wm, wn;
    uint32_t aoff[2], boff[2], lbase;
    Job j;
    i32x4 sa, sb;
    uint32_t va[2], vb[2];
    int nk, head;

    // a partial last K tile comes first
    __device__ __forceinline__ int k0_of(int q) const {
        return (head ? (q == 0 ? nk - 1 : q - 1) : q) * C::BK;
    }
    // column of LDS row lr of B (bf16 output: a lane's two fragments of 32
    // columns hold eight consecutive ones)
    __device__ __forceinline__ static int b_col(int lr) {
        const int p = lr & 31;
        return (lr & ~31) +
               (C::CBF16 ? 8 * ((p >> 2) & 3) + 4 * (p >> 4) + (p & 3) : p);
    }
    __device__ __forceinline__ void init(char *s) {
        smem = s;
        tid = threadIdx.x;
        lane = tid & 63;
        wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        lbase = lds_addr(s) + wave * 1024;
        wm = wave >> 1;
        wn = wave & 1;
        const int r = lane & 15, grp = lane >> 4;
        const uint32_t base = lds_addr(s);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int ch = FA::F8 || MIX ? 2 * grp + q : 4 * q + grp;
            const int c = (ch ^ ph_swz(r)) << 4;
            aoff[q] = base + (wm * 32 + r) * 128 + c;
            boff[q] = base + ABYTES + (wn * 64 + r) * 128 + c;
        }
        if constexpr (MIX)
            boff[0] = base + ABYTES + (wn * 64 + r) * 64 +
                      ((grp ^ ((r >> 2) & 3)) << 4);
    }
    // row and 16-byte chunk of K that lane l loads in 1 KiB block `blk`
    __device__ __forceinline__ int a_row(int i) const {
        return (i * 8 + wave) * 8 + (lane >> 3);
    }
    __device__ __forceinline__ int a_chunk(int i) const {
        return (lane & 7) ^ ph_swz(a_row(i));
    }
    __device__ __forceinline__ int mb_row() const {       // MIX: B
        return wave * 16 + (lane >> 2);
    }
    __device__ __forceinline__ int mb_chunk() const {
        return (lane & 3) ^ ((mb_row() >> 2) & 3);
    }
    __device__ __forceinline__ void set_job(const Job &nj) {
        j = nj;
        j.K = __builtin_amdgcn_readfirstlane(j.K);
        nk = (j.K + C::BK - 1) / C::BK;
        head = j.K % C::BK ? 1 : 0;
        sa = make_srd(j.a_row, sat_bytes(j.a_rem));
        sb = make_srd(j.b_row, sat_bytes(j.b_rem));
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            va[i] = (uint32_t)((a_row(i) * j.lda + a_chunk(i) * C::EPC) *
                               C::ES);
            if constexpr (MIX) {
                vb[i] = (uint32_t)(b_col(mb_row()) * j.ldb + mb_chunk() * 16);
            } else {
                vb[i] = (uint32_t)((b_col(a_row(i)) * j.ldb +
                                    a_chunk(i) * C::EPC) * C::ES);
            }
        }
    }
    __device__ __forceinline__ void load_b(uint32_t stage,
                                           const uint32_t (&v)[2], int so) {
        if constexpr (MIX)
            ph_dma1<ABYTES>(sb, lbase + stage, v[0], so);
        else
            ph_dma2<ABYTES>(sb, lbase + stage, v, so);
    }
    // A's and B's share of sequence tile q into its stage.  In tile 0,
    // possibly K's tail, chunks not wholly inside K load as zeros.
    __device__ __forceinline__ void issue_a(int q) {
        ph_dma2<0>(sa, lbase + (q & 3) * STG, va, k0_of(q) * C::ES);
    }
    __device__ __forceinline__ void issue_b(int q) {
        load_b((q & 3) * STG, vb, k0_of(q) * BES);
    }
    __device__ __forceinline__ void issue_tile0() {
        const int k0 = k0_of(0);
        uint32_t w[2], u[2] = {vb[0], vb[1]};
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const bool in = k0 + (a_chunk(i) + 1) * C::EPC <= j.K;
            w[i] = in ? va[i] : kOutOfRange;
            if constexpr (!MIX)
                u[i] = in ? vb[i] : kOutOfRange;
        }
        if constexpr (MIX)
            if (k0 + (mb_chunk() + 1) * 16 > j.K) u[0] = kOutOfRange;
        ph_dma2<0>(sa, lbase, w, k0 * C::ES);
        load_b(0, u, k0 * BES);
    }
    __device__ __forceinline__ void issue_first() {
        if (nk > 0) issue_tile0();
#pragma unroll
        for (int q = 1; q < 3; ++q)
            if (q < nk) {
                issue_a(q);
                issue_b(q);
            }
    }
    // The chunk that straddles K was loaded as zeros: its K % EPC valid
    // elements of every row, one by one (MIX: K is whole chunks of both).
    __device__ __forceinline__ void fill_tail() {
        const int rem = j.K % C::EPC, kbase = j.K - rem;
        const int chunk = (kbase - k0_of(0)) / C::EPC;
        auto put = [&](char *dst, const char *src, bool ok) {
            for (int e = 0; e < rem * C::ES; ++e) dst[e] = ok ? src[e] : 0;
        };
        for (int lr = tid; lr < 128; lr += C::THREADS)
            put(smem + lr * 128 + ((chunk ^ ph_swz(lr)) << 4),
                j.a + ((int64_t)(j.m0 + lr) * j.lda + kbase) * C::ES,
                j.m0 + lr < j.M);
        for (int lr = tid; lr < 128; lr += C::THREADS)
            put(smem + ABYTES + lr * 128 + ((chunk ^ ph_swz(lr)) << 4),
                j.b + ((int64_t)(j.n0 + b_col(lr)) * j.ldb + kbase) * C::ES,
                j.n0 + b_col(lr) < j.N);
    }
    __device__ __forceinline__ static i32x4 ld(uint32_t p) {
        return *reinterpret_cast<const lds_i32x4 *>(p);
    }
    template <int NF>
    __device__ __forceinline__ static void read_rows(PhFrag<C, NF> &o,
                                                     uint32_t p0,
                                                     uint32_t p1) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const i32x4 lo = ld(p0 + f * 2048), hi = ld(p1 + f * 2048);
            if constexpr (FA::F8) {
                o.v[f][0] = i32x8{lo[0], lo[1], lo[2], lo[3],
                                  hi[0], hi[1], hi[2], hi[3]};
            } else {
                o.v[f][0] = lo;
                o.v[f][1] = hi;
            }
        }
    }
    __device__ __forceinline__ void read(FA &a, FB &b, uint32_t stage) const {
        read_rows(a, aoff[0] + stage, aoff[1] + stage);
        if constexpr (MIX) {      // codes, see decode()
#pragma unroll
            for (int f = 0; f < 4; ++f)
                b.v[f][0] = ld(boff[0] + stage + f * 1024);
        } else {
            read_rows(b, boff[0] + stage, boff[1] + stage);
        }
    }
    __device__ __forceinline__ static void decode(FB &b) {
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            const i32x4 w = b.v[f][0];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const uint2 lo = e4m3x4_to_bf16x4(w[2 * q]);
                const uint2 hi = e4m3x4_to_bf16x4(w[2 * q + 1]);
                b.v[f][q] = i32x4{(int)lo.x, (int)lo.y, (int)hi.x, (int)hi.y};
            }
        }
    }

    template <class P>
    __device__ __forceinline__ void run(const P &prov, char *s) {
        const int G = prov.n_prog(), total = prov.count();
        int t = program_slot(blockIdx.x, G);
        if (t >= total) return;
        init(s);
        int njob = 0;
        Acc acc;
        FA a;
        FB b;
        set_job(prov.job(t));
        tg::issue_scales<C>(j, scale_slot<C>(smem, 0), wave, lane);
        issue_first();
        while (true) {
#pragma unroll
            for (int i = 0; i < 8; ++i) mfma_zero(acc[i >> 2][i & 3]);
            wait_vmem();      // also the previous sub-tensor's stores
            slot_end();
            if (!MIX && j.K % C::EPC != 0) {
                fill_tail();
                __syncthreads();
            }
            if (wave >> 2) slot_end();        // one slot behind
#pragma unroll 1
            for (int q = 0; q < nk; ++q) {
                // Memory slot.  The stage loaded into was last read by the
                // group behind in the slot before, which ended after its
                // data had arrived.
                read(a, b, (q & 3) * STG);
                const bool more_k = q + 3 < nk;
                if (more_k) issue_a(q + 3);
                // the next tile has landed (B's loads of tile q + 3 come in
                // the compute slot)
                const int after = nk - 2 - q;
                if (__builtin_expect(after >= 2, 1)) wait_vmem_le<LOADS + 2>();
                else if (after == 1) wait_vmem_le<LOADS>();
                else wait_vmem();
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                if constexpr (MIX) decode(b);
                slot_end();
                __builtin_amdgcn_s_setprio(1);
                if (more_k) issue_b(q + 3);
                // (decoded fragments are vector-ALU results)
                if constexpr (MIX) asm volatile("s_nop 1" ::: "memory");
#pragma unroll
                for (int h = 0; h < NQ; ++h)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int f = 0; f < 4; ++f)
                            ph_mfma<C>(a.v[i][h], b.v[f][h], acc[i][f]);
                __builtin_amdgcn_s_setprio(0);
                slot_end();
            }
            if (!(wave >> 2)) slot_end();     // level again: LDS is free
            mfma_drain();
            t += G;
            const bool more = t < total;
            const Job done = j;
            if (more) {
                set_job(prov.job(t));
                tg::issue_scales<C>(j, scale_slot<C>(smem, njob + 1), wave,
                                    lane);
                issue_first();
            }
            if (done.scale_a || done.scale_b)
                Store::template store<true>(done, acc,
                                            scale_slot<C>(smem, njob), smem,
                                            lane, wave);
            else
                Store::template store<false>(done, acc, nullptr, smem, lane,
                                             wave);
            if (!more) break;
            ++njob;
        }
    }
};

template <class C>
__global__ __launch_bounds__(512)
__attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_phased128_kernel(
    GemmArgs g) {
    extern __shared__ __align__(1024) char smem[];
    SingleProvider<C> p{g};
    Phased128<C> k;
    k.run(p, smem);
}

template <class C>
__global__ __launch_bounds__(512)
__attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_phased128_grouped_kernel(
    const GroupProblem *__restrict__ tab, int n, int total, int G) {
    extern __shared__ __align__(1024) char smem[];
    GroupProvider<C> p{tab, n, total, G};
    Phased128<C> k;
    k.run(p, smem);
}

template <int DT, bool CBF16>
VariantEntry entry128() {
    typedef Cfg<DT, 128, 128, 4, 2, true, CBF16, 128, 4, TG_SCHED_LOCKSTEP> C;
    VariantEntry e{};
    e.v.dtype = DT;
    e.v.bm = C::BM; e.v.bn = C::BN; e.v.bk = C::BK; e.v.stages = C::NS;
    e.v.sched = TG_SCHED_LOCKSTEP;
    e.v.wm = C::WM; e.v.wn = C::WN;
    e.v.b_nk = true; e.v.c_bf16 = CBF16;
    e.kernel = reinterpret_cast<const void *>(&gemm_phased128_kernel<C>);
    if constexpr (DT == TG_BF16)
        e.grouped =
            reinterpret_cast<const void *>(&gemm_phased128_grouped_kernel<C>);
    e.threads = C::THREADS;
    e.smem = Phased128<C>::SMEM;
    return e;
}

// bf16 by e4m3: one block of 2 x 2 sub-tensors of 64 x 64 per program.
template <class C>
struct MixedProvider {
    const SimpleArgs &g;
    __device__ int n_prog() const { return g.n_prog; }
    __device__ int count() const { return g.n_prog; }
    __device__ Job job(int) const {
        int bm, bn;
        simple_block(blockIdx.x, g.n_prog, g.blocks_m, bm, bn);
        Job j;
        j.a = static_cast<const char *>(g.a);
        j.b = static_cast<const char *>(g.b);
        j.c = g.c;
        j.scale_a = g.scale_a; j.scale_b = g.scale_b;
        j.wcount = g.wcount;
        j.lda = g.lda; j.ldb = g.ldb; j.ldc = g.ldc;
        j.M = g.M; j.N = g.N; j.K = g.K;
        j.m0 = bm * 128; j.n0 = bn * 128;
        j.a_row = j.a + (int64_t)j.m0 * j.lda * 2;
        j.a_rem = (int64_t)(j.M - j.m0) * j.lda * 2;
        j.b_row = j.b + (int64_t)j.n0 * j.ldb;
        j.b_rem = (int64_t)(j.N - j.n0) * j.ldb;
        return j;
    }
};

template <class C>
__global__ __launch_bounds__(512)
__attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_mixed128_kernel(
    SimpleArgs g) {
    extern __shared__ __align__(1024) char smem[];
    MixedProvider<C> p{g};
    Phased128<C, true> k;
    k.run(p, smem);
}

template <bool CBF16>
hipError_t launch_mixed_out(const SimpleArgs &a, hipStream_t st) {
    typedef Cfg<TG_BF16, 128, 128, 4, 2, true, CBF16, 128, 4,
                TG_SCHED_LOCKSTEP> C;
    constexpr int lds = Phased128<C, true>::SMEM;
    static LdsRequest request;
    const hipError_t ready = request(
        {reinterpret_cast<const void *>(&gemm_mixed128_kernel<C>)}, lds);
    if (ready != hipSuccess) return ready;
    hipLaunchKernelGGL(gemm_mixed128_kernel<C>, dim3((unsigned)a.n_prog),
                       dim3(C::THREADS), lds, st, a);
    return hipGetLastError();
}

template <int DT, bool BNK, bool CBF16>
VariantEntry entry(int sched = TG_SCHED_CROSS) {
    typedef Cfg<DT, 256, 256, 2, 4, BNK, CBF16, 128, 2, TG_SCHED_CROSS> C;
    VariantEntry e{};
    e.v.dtype = DT;
    e.v.bm = C::BM; e.v.bn = C::BN; e.v.bk = C::BK; e.v.stages = C::NS;
    e.v.sched = sched;
    e.v.wm = C::WM; e.v.wn = C::WN;
    e.v.b_nk = BNK; e.v.c_bf16 = CBF16;
    e.kernel = reinterpret_cast<const void *>(&gemm_phased_kernel<C, false>);
    if constexpr (DT == TG_BF16) {
        e.planes =
            reinterpret_cast<const void *>(&gemm_phased_kernel<C, true>);
        e.grouped =
            reinterpret_cast<const void *>(&gemm_phased_grouped_kernel<C>);
    }
    e.threads = C::THREADS;
    e.smem = Phased<C>::SMEM;
    return e;
}

}  // namespace

// The two-stage cross-tile configurations.  TG_SCHED_CROSS_WARM, which
// callers, tuning files and the long-K default name, runs the same kernel:
// its loads run far enough ahead that an L2 warm-up has nothing to hide
// (4096^2 x 32768: 747 us, 927 with the warm-up on the cross-tile ring).
const VariantEntry *phased_entries(int *n) {
    static const VariantEntry e[] = {
        entry<TG_BF16, true, false>(),  entry<TG_BF16, true, true>(),
        entry<TG_BF16, false, false>(), entry<TG_BF16, false, true>(),
        entry<TG_FP8_E4M3, true, false>(), entry<TG_FP8_E4M3, true, true>(),
        entry<TG_BF16, true, false>(TG_SCHED_CROSS_WARM),
        entry<TG_BF16, true, true>(TG_SCHED_CROSS_WARM),
        entry128<TG_BF16, false>(), entry128<TG_BF16, true>(),
        entry128<TG_FP8_E4M3, false>(), entry128<TG_FP8_E4M3, true>(),
    };
    *n = (int)(sizeof e / sizeof e[0]);
    return e;
}

// (checked on the host: blocks of 128 x 128, aligned rows, K of whole chunks
// of both operands, offsets below 2^31 within a block)
hipError_t launch_mixed(const SimpleArgs &a, hipStream_t st) {
    return a.c_bf16 ? launch_mixed_out<true>(a, st)
                    : launch_mixed_out<false>(a, st);
}

}  // namespace tg
