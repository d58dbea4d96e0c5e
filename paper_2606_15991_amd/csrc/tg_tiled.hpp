// tg_tiled.hpp -- what the tiled kernel sources share: the configuration of an
// instantiation, LDS layouts, direct loads, the epilogue, and the providers
// of a program's owned sub-tensors.
#pragma once

#include "tg_device.hpp"
#include "tg_internal.hpp"

namespace tg {
// One compiled instantiation and its kernels.
struct VariantEntry {
    TiledVariant v;
    const void *kernel;
    const void *grouped = nullptr;  // bf16 only (grouped launches take no other)
    int threads;
    int smem;
    const void *planes = nullptr;   // products of planes (GemmArgs::kp)
};

// The phased schedule's entries (gemm_phased.hip).
const VariantEntry *phased_entries(int *count);

namespace {

typedef __attribute__((address_space(3))) void lds_void;
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

template <int DT>
struct DtypeTraits;
template <>
struct DtypeTraits<TG_BF16> {
    static constexpr int ES = 2;
};
template <>
struct DtypeTraits<TG_F32> {
    static constexpr int ES = 4;
};
template <>
struct DtypeTraits<TG_FP8_E4M3> {
    static constexpr int ES = 1;
};

template <int DT, int BM_, int BN_, int WM_, int WN_, bool BNK_, bool CBF16_,
          int RBY_ = 128, int NS_ = 2, int SCH_ = TG_SCHED_LOCKSTEP>
struct Cfg {
    static constexpr int DTYPE = DT;
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_;
    static constexpr bool BNK = BNK_, CBF16 = CBF16_;
    static constexpr int ES = DtypeTraits<DT>::ES;
    static constexpr int EPC = 16 / ES;         // elements per 16-byte chunk
    static constexpr int RBY = RBY_;            // bytes of K per operand row
    static constexpr int NS = NS_;              // LDS stages in the ring
    static constexpr int SCHED = SCH_;          // wavefront schedule
    static constexpr bool PP = SCH_ == TG_SCHED_PINGPONG;
    static constexpr bool XT = SCH_ == TG_SCHED_CROSS;
    static constexpr bool STG = SCH_ == TG_SCHED_STAGED;
    static constexpr bool BLK = SCH_ == TG_SCHED_BULK;
    static constexpr int BK = RBY / ES;         // K elements per K tile
    static constexpr int CPRW = RBY / 16;       // 16-byte chunks per row
    static constexpr int RPK = 1024 / RBY;      // rows per 1 KiB block
    static constexpr int NW = WM * WN;          // wavefronts
    static constexpr int THREADS = NW * 64;
    static constexpr int TM = BM / WM, TN = BN / WN;
    static constexpr int FM = TM / 32, FN = TN / 32;
    static constexpr bool B_KMAJOR = !BNK && ES >= 2;  // [BK][BN] in LDS
    static constexpr int RB = BN * ES;          // bytes per k-major B row
    static constexpr int CPR = RB / 16;         // chunks per k-major B row
    static constexpr int STAGE = (BM + BN) * RBY;   // bytes per LDS stage
    // Per-row and per-column scales of an owned sub-tensor live in LDS next
    // to the stages, one slot per sub-tensor in flight (NS + 1 slots: the
    // loads run at most NS - 1 K tiles, hence sub-tensors, ahead).
    static constexpr int SCALE_SLOT = (BM + BN) * 4;
    static constexpr int NSLOT = NS + 1;
    static constexpr int SMEM =
        (XT && NS == 3 ? 5 * (STAGE / 2) : NS * STAGE) +
        (!XT && SCH_ != TG_SCHED_STAGED &&
                 SCH_ != TG_SCHED_BULK
             ? NSLOT * SCALE_SLOT
             : 0);
    static constexpr int LPW = STAGE / 1024 / NW;   // 1 KiB loads per wave
    static_assert(TM % 32 == 0 && TN % 32 == 0, "wave tile");
    static_assert(RBY == 128 || RBY == 64, "K-tile row bytes");
    static_assert(NS == 2 || NS == 4 ||
                      (NS == 5 && XT && RBY == 64) ||
                      (NS == 5 && SCH_ == TG_SCHED_BULK) ||
                      (NS == 3 && XT && RBY == 128 &&
                       BM == BN),
                  "ring of 2 or 4 stages, 5 of 64-byte rows, or 5 operand "
                  "halves (NS = 3)");
    // NS = 3 with the cross-tile schedule: the LDS holds five operand
    // tiles (A or B of one K tile each) instead of three whole stages.
    static constexpr bool HALVES = XT && NS == 3;
    static_assert((BM / RPK) % NW == 0, "A 1 KiB blocks per wave");
    static_assert(B_KMAJOR ? (BK * RB / 1024) % NW == 0
                           : (BN / RPK) % NW == 0, "B 1 KiB blocks per wave");
    static_assert(BNK || DT != TG_FP8_E4M3, "e4m3 B must be stored N x K");
    static_assert(!B_KMAJOR || CPR >= 4, "k-major B rows of >= 64 bytes");
    static_assert(DT != TG_FP8_E4M3 || BK >= 64, "e4m3 K tile >= 64");
    static_assert(LPW * (NS - 1) < 64, "vmcnt range");
    // Wavefronts per SIMD when LDS limits the workgroups per CU (160 KiB):
    // the register budget and scheduling target of the compiler.  Without
    // it the scheduler aims at a higher occupancy than LDS allows and
    // trades the fragment double buffer for fewer registers.
    static constexpr int WG_PER_CU_ = 163840 / SMEM;
    static constexpr int WPE_ = WG_PER_CU_ * NW / 4;
    static constexpr int WPE_MAX_ = 4;
    static constexpr int WPE = WPE_ < 1 ? 1 : (WPE_ > WPE_MAX_ ? WPE_MAX_ : WPE_);
    static_assert(!PP || (WM == 2 && NW == 8 && NS >= 3),
                  "ping-pong: two groups of four wavefronts, >= 3 stages");
    static_assert(!XT || ES <= 2, "cross-tile schedule: bf16 or e4m3");
    static_assert(!BLK || (DT == TG_BF16 && BNK && NS >= 4 &&
                           BK / 16 * (FM + FN) * 4 <= 128),
                  "bulk schedule: bf16, B stored N x K, a ring of at least "
                  "four stages, one K tile of fragments in 64 registers");
    static_assert(!STG || (DT == TG_BF16 && BNK && RBY == 128 && NS == 2),
                  "staged schedule: bf16, B stored N x K, 64-deep K tiles, "
                  "two LDS stages");
};

// Row-major [rows][RBY bytes] operand stage: chunk c of row r sits at chunk
// position c ^ f(r), with f(r) = (r >> 1) & 7 for 128-byte rows and
// ((r >> 1) ^ (r >> 3)) & 3 for 64-byte rows.  Any 16 consecutive rows read
// at one logical chunk then cover 16 distinct 16-byte bank groups of a
// 256-byte bank window (and any 8 of them 8 groups of a 128-byte window), so
// the 16-byte fragment reads are conflict-free.  f is unchanged by a shift
// of 32 rows, so the fragments of one K step, 32 rows apart, sit at one lane
// offset plus constants.
template <class C>
__device__ __forceinline__ int swz_f(int row) {
    if constexpr (C::RBY == 128)
        return (row >> 1) & 7;
    else
        return ((row >> 1) ^ (row >> 3)) & 3;
}
template <class C>
__device__ __forceinline__ int swz(int row, int chunk) {
    return row * C::RBY + ((chunk ^ swz_f<C>(row)) << 4);
}

// Chunk permutation of k-major B rows, by k & 3: the four rows of a 16-lane
// transposing read (and of two such groups read together) land in distinct
// 16-byte bank groups.
template <class C>
__device__ __forceinline__ int swz_kmajor(int k) {
    if constexpr (C::ES == 4) return 0;   // binary32: plain dword reads
    if constexpr (C::CPR >= 16) {
        constexpr uint32_t tab = 0u | (4u << 8) | (10u << 16) | (14u << 24);
        return (tab >> (8 * (k & 3))) & 0xff;
    } else if constexpr (C::CPR == 8) {
        return 2 * (k & 3);
    } else {
        return 2 * (k & 1);
    }
}

// Vector-memory counter waits, as s_waitcnt instructions the compiler sees
// (its own wait insertion then knows which loads are complete).  Encoding:
// vmcnt in bits [3:0] and [15:14], expcnt [6:4] and lgkmcnt [11:8] at their
// no-wait maxima.
template <int N>
__device__ __forceinline__ void wait_vmem_le() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) |
                               (15 << 8));
}

__device__ __forceinline__ void wait_vmem() { wait_vmem_le<0>(); }

// Workgroup barrier for the K-tile ring.  __syncthreads() carries a
// workgroup-scope fence, which waits for every outstanding global access of
// the wavefront, including the loads of later K tiles that must stay in
// flight.  The ring needs less: this wavefront's LDS reads are complete (so
// a stage may be overwritten after the barrier) and the loads of the tile
// about to be read have landed (waited for by the caller).
__device__ __forceinline__ void ring_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// One owned sub-tensor as the kernels see it.
struct Job {
    const char *a;
    const char *b;
    void *c;
    const float *scale_a;
    const float *scale_b;
    int32_t *wcount;
    int64_t lda, ldb, ldc;
    int32_t M, N, K;
    int32_t m0, n0;
    // Load streams of the sub-tensor, fixed for all its K tiles: first
    // byte of its A rows (and of its B rows, or of its B columns in row 0
    // for B stored K x N) and the bytes from there to the operand's end.
    const char *a_row, *b_row;
    int64_t a_rem, b_rem;
};

// ------------------------------------------------------------ tile loads

// Buffer resource of `bytes` bytes at `base` (raw buffer, no stride).
// Lanes whose offset is at or beyond `bytes` read zeros; the direct load
// then writes those zeros into LDS.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *base,
                                                           uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base),
                                             (short)0, (int)bytes,
                                             0x00020000);
}

constexpr uint32_t kOutOfRange = 0x80000000u;

// Direct loads are issued from inline assembly.  The compiler's own
// dependency tracking would place waits on the vector-memory counter in
// front of LDS reads it cannot prove disjoint from a load's LDS
// destination, which drains the loads that must stay in flight; the K-tile
// schedules here order every LDS access explicitly instead (counter waits
// before workgroup barriers).
//
// Descriptor words of a raw buffer (no stride) in scalar registers.
__device__ __forceinline__ i32x4 make_srd(const void *base, uint32_t bytes) {
    const uint64_t p = reinterpret_cast<uint64_t>(base);
    i32x4 d;
    d[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)p);
    d[1] = __builtin_amdgcn_readfirstlane((int)((uint32_t)(p >> 32) & 0xffffu));
    d[2] = __builtin_amdgcn_readfirstlane((int)bytes);
    d[3] = 0x00020000;
    return d;
}

// LDS address of a generic pointer into the workgroup's LDS: its low 32
// bits (the shared aperture occupies the high half of the flat address).
// Taken directly rather than through an address-space cast, which would
// add a null-pointer test to every load.
__device__ __forceinline__ uint32_t lds_addr(const char *p) {
    return __builtin_amdgcn_readfirstlane(
        (int)static_cast<uint32_t>(reinterpret_cast<uintptr_t>(p)));
}

// One 16-byte-per-lane load from buffer `srd` at byte offset `voff` into
// LDS at dst + 16 * lane.  M0 holds the LDS address; one wait state
// separates its write from the load.  The first load after `srd` was
// formed also waits five states, the distance a vector-ALU write of a
// scalar register needs before a vector-memory instruction reads it.
template <bool FIRST>
__device__ __forceinline__ void dma16(const i32x4 &srd, char *dst,
                                      uint32_t voff) {
    const uint32_t lds = lds_addr(dst);
    if constexpr (FIRST)
        asm volatile(
            "s_nop 4\n\ts_mov_b32 m0, %0\n\ts_nop 0\n\t"
            "buffer_load_dwordx4 %1, %2, 0 offen lds"
            :
            : "s"(lds), "v"(voff), "s"(srd)
            : "memory", "m0");
    else
        asm volatile(
            "s_mov_b32 m0, %0\n\ts_nop 0\n\t"
            "buffer_load_dwordx4 %1, %2, 0 offen lds"
            :
            : "s"(lds), "v"(voff), "s"(srd)
            : "memory", "m0");
}

// One 4-byte-per-lane load into LDS at dst + 4 * lane (same protocol as
// dma16).
__device__ __forceinline__ void dma4(const i32x4 &srd, char *dst,
                                     uint32_t voff) {
    const uint32_t lds = lds_addr(dst);
    asm volatile(
        "s_nop 4\n\ts_mov_b32 m0, %0\n\ts_nop 0\n\t"
        "buffer_load_dword %1, %2, 0 offen lds"
        :
        : "s"(lds), "v"(voff), "s"(srd)
        : "memory", "m0");
}

__device__ __forceinline__ uint32_t sat_bytes(int64_t b) {
    return b <= 0 ? 0u : (b >= 0x7fffffff ? 0x7fffffffu : (uint32_t)b);
}

template <class C>
__device__ __forceinline__ void set_streams(Job &j) {
    j.a_row = j.a + (int64_t)j.m0 * j.lda * C::ES;
    j.a_rem = (int64_t)(j.M - j.m0) * j.lda * C::ES;
    if constexpr (C::B_KMAJOR) {
        j.b_row = j.b + (int64_t)j.n0 * C::ES;
        j.b_rem = ((int64_t)j.K * j.ldb - j.n0) * C::ES;
    } else {
        j.b_row = j.b + (int64_t)j.n0 * j.ldb * C::ES;
        j.b_rem = (int64_t)(j.N - j.n0) * j.ldb * C::ES;
    }
}

// Direct HBM -> LDS issue of K tile k0 of one owned sub-tensor.  Each lane
// fetches the 16-byte chunk that the LDS swizzle places at its position:
// lane l of the 1 KiB block rb writes row rb * RPK + l / CPRW at chunk
// position l % CPRW, which holds logical chunk (l % CPRW) ^ f(row).  Rows
// beyond M / N and chunks not wholly inside K read as zeros (out-of-range
// buffer offsets); a chunk straddling K is filled by fill_k_tail.
template <class C, int ROWS>
__device__ __forceinline__ void issue_operand(const char *row0, int64_t rem,
                                              int64_t ld, int k0, int K,
                                              char *dst, int wave, int lane) {
    const int64_t skip = (int64_t)k0 * C::ES;
    const i32x4 srd = make_srd(row0 + skip, sat_bytes(rem - skip));
    const int rsub = lane / C::CPRW, p = lane % C::CPRW;
#pragma unroll
    for (int i = 0; i < ROWS / C::RPK / C::NW; ++i) {
        const int rb = i * C::NW + wave;
        const int row = rb * C::RPK + rsub;           // row within the tile
        const int kc = p ^ swz_f<C>(row);
        const bool kin = k0 + (kc + 1) * C::EPC <= K;
        const uint32_t off = kin ? (uint32_t)((row * ld + kc * C::EPC) * C::ES)
                                 : kOutOfRange;
        if (i == 0)
            dma16<true>(srd, dst + rb * 1024, off);
        else
            dma16<false>(srd, dst + rb * 1024, off);
    }
}

// The A tile of K tile k0 into As.
template <class C>
__device__ __forceinline__ void issue_a(const Job &j, char *As, int k0,
                                        int wave, int lane) {
    issue_operand<C, C::BM>(j.a_row, j.a_rem, j.lda, k0, j.K, As, wave,
                            lane);
}

// The B tile of K tile k0 into Bs.
template <class C>
__device__ __forceinline__ void issue_b(const Job &j, char *Bs, int k0,
                                        int wave, int lane) {
    if constexpr (!C::B_KMAJOR) {
        issue_operand<C, C::BN>(j.b_row, j.b_rem, j.ldb, k0, j.K, Bs,
                                wave, lane);
    } else {
        // k-major B: descriptor from (k0, n0); rows k >= K are past its end,
        // columns >= N are masked per lane
        const int64_t skip = (int64_t)k0 * j.ldb * C::ES;
        const i32x4 srd = make_srd(j.b_row + skip, sat_bytes(j.b_rem - skip));
#pragma unroll
        for (int i = 0; i < C::BK * C::RB / 1024 / C::NW; ++i) {
            const int gi = i * C::NW + wave;
            const int off = gi * 1024 + lane * 16;
            const int k = off / C::RB;
            const int lc = ((off % C::RB) >> 4) ^ swz_kmajor<C>(k);
            const bool nin = j.n0 + lc * C::EPC < j.N;
            const uint32_t voff =
                nin ? (uint32_t)((k * j.ldb + lc * C::EPC) * C::ES)
                    : kOutOfRange;
            if (i == 0)
                dma16<true>(srd, Bs + gi * 1024, voff);
            else
                dma16<false>(srd, Bs + gi * 1024, voff);
        }
    }
}

// parts: bit 0 = the A tile, bit 1 = the B tile, into one stage.
template <class C>
__device__ __forceinline__ void issue_direct(const Job &j, char *stage,
                                             int k0, int wave, int lane,
                                             int parts = 3) {
    if (parts & 1) issue_a<C>(j, stage, k0, wave, lane);
    if (parts & 2) issue_b<C>(j, stage + C::BM * C::RBY, k0, wave, lane);
}

// Scales of one owned sub-tensor into its LDS slot: scale_a[m0 .. m0+BM)
// then scale_b[n0 .. n0+BN), 64 per instruction, instructions dealt out
// over the wavefronts.  Entries beyond M / N load as zeros.
template <class C>
__device__ __forceinline__ void issue_scales(const Job &j, char *slot,
                                             int wave, int lane) {
    constexpr int IA = (C::BM + 63) / 64, IB = (C::BN + 63) / 64;
    if (j.scale_a) {
        const i32x4 srd = make_srd(j.scale_a + j.m0, sat_bytes((int64_t)(j.M - j.m0) * 4));
#pragma unroll
        for (int i = 0; i < IA; ++i)
            if (i % C::NW == wave) {
                const int r = i * 64 + lane;
                dma4(srd, slot + i * 256, r < C::BM ? (uint32_t)(r * 4) : kOutOfRange);
            }
    }
    if (j.scale_b) {
        const i32x4 srd = make_srd(j.scale_b + j.n0, sat_bytes((int64_t)(j.N - j.n0) * 4));
#pragma unroll
        for (int i = 0; i < IB; ++i)
            if ((IA + i) % C::NW == wave) {
                const int c = i * 64 + lane;
                dma4(srd, slot + C::BM * 4 + i * 256,
                     c < C::BN ? (uint32_t)(c * 4) : kOutOfRange);
            }
    }
}

// LDS scale slot of the n-th owned sub-tensor of a program.
template <class C>
__device__ __forceinline__ char *scale_slot(char *smem, int n) {
    return smem + C::NS * C::STAGE + (n % C::NSLOT) * C::SCALE_SLOT;
}

// B operand of the 32x32x16 bf16 instruction from a k-major B stage:
// two transposing reads.  In each 16-lane group, lane r names row
// k = kb + r / 4 at columns c0 + 4 (r % 4) .. +3, and lane i of the group
// receives column c0 + i at rows kb .. kb + 3.
template <class C>
__device__ __forceinline__ i32x4 read_b_kmajor(const char *Bs, int kk,
                                               int col0, int lane) {
    const int g = lane >> 4, r = lane & 15;
    const int half = g >> 1, cg = g & 1;
    const int n = col0 + cg * 16 + 4 * (r & 3);
    i32x4 out;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int k = kk * 16 + half * 8 + q * 4 + (r >> 2);
        const char *p = Bs + k * C::RB +
                        (((n >> 3) ^ swz_kmajor<C>(k)) << 4) + ((n & 7) << 1);
        const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_s16x4 *)(p));
        const uint32_t v0 = (uint16_t)v[0], v1 = (uint16_t)v[1];
        const uint32_t v2 = (uint16_t)v[2], v3 = (uint16_t)v[3];
        out[2 * q] = (int)(v0 | (v1 << 16));
        out[2 * q + 1] = (int)(v2 | (v3 << 16));
    }
    return out;
}

// Store one program's accumulators into its own sub-tensor.
// 32 x 32 MFMA result layout: lane l, register v holds
//   row 8 * (v / 4) + 4 * (l / 32) + v % 4,  column l % 32.
// Stores go through a buffer descriptor rooted at the sub-tensor's first
// element with 32-bit offsets; elements outside the output (rows >= M,
// columns >= N) get an out-of-range offset, which the hardware drops.
// `scl`: this sub-tensor's scale slot in LDS (direct-load programs), or
// nullptr to read the scales from global memory.
template <class C>
__device__ __forceinline__ void epilogue(const Job &j, int wm, int wn,
                                         int lane,
                                         f32x16 (&acc)[C::FM][C::FN],
                                         const char *scl) {
    constexpr int OES = C::CBF16 ? 2 : 4;
    // The address arithmetic below is loop-invariant in a persistent
    // program; hidden from the optimiser so that it is formed here, per
    // stored sub-tensor, instead of being hoisted and held in registers
    // across the whole K loop.
    int lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)j.ldc);
    int hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)(j.ldc >> 32));
    asm volatile("" : "+s"(lo), "+s"(hi));
    const int64_t ldc = (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
    const int col_l = lane & 31, half = lane >> 5;
    const int r0 = wm * C::TM + 4 * half;        // row of v = 0, i = 0
    const int c0 = wn * C::TN + col_l;           // column of jj = 0
    char *base = static_cast<char *>(j.c) +
                 ((int64_t)j.m0 * ldc + j.n0) * OES;
    const __amdgpu_buffer_rsrc_t r = make_rsrc(
        base, sat_bytes(((int64_t)(j.M - j.m0 - 1) * ldc + (j.N - j.n0)) *
                        OES));
    const int rows_left = j.M - j.m0 - r0;       // rows with local index < this
    const int cols_left = j.N - j.n0 - c0;
    // Scales are loaded, and waited for, before any store is issued, and
    // inside the branch that loads them, so that no load of this epilogue
    // is outstanding (or believed outstanding) when the K loop resumes.
    const float *lsa = reinterpret_cast<const float *>(scl);
    const float *lsb = lsa + C::BM;
    float sb[C::FN];
#pragma unroll
    for (int jj = 0; jj < C::FN; ++jj) sb[jj] = 1.0f;
    if (j.scale_b) {
        if (scl) {
#pragma unroll
            for (int jj = 0; jj < C::FN; ++jj) sb[jj] = lsb[c0 + jj * 32];
        } else {
#pragma unroll
            for (int jj = 0; jj < C::FN; ++jj)
                if (jj * 32 < cols_left)
                    sb[jj] = j.scale_b[j.n0 + c0 + jj * 32];
            wait_vmem();
        }
    }
    const uint32_t lane_off = (uint32_t)((r0 * ldc + c0) * OES);
    auto store_rows = [&](int i, const float (&sa)[16]) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int dr = i * 32 + 8 * (v >> 2) + (v & 3);
            const bool row_ok = dr < rows_left;
            const uint32_t roff = lane_off + (uint32_t)(dr * ldc * OES);
#pragma unroll
            for (int jj = 0; jj < C::FN; ++jj) {
                const bool ok = row_ok && jj * 32 < cols_left;
                const uint32_t off = ok ? roff + jj * 32 * OES : kOutOfRange;
                const float x = acc[i][jj][v] * sb[jj] * sa[v];
                if constexpr (C::CBF16)
                    __builtin_amdgcn_raw_buffer_store_b16(
                        (unsigned short)f32_to_bf16_bits(x), r, off, 0, 0);
                else
                    __builtin_amdgcn_raw_buffer_store_b32(
                        __builtin_bit_cast(uint32_t, x), r, off, 0, 0);
            }
        }
    };
    if (!j.scale_a) {
        const float ones[16] = {1.f, 1.f, 1.f, 1.f, 1.f, 1.f, 1.f, 1.f,
                                1.f, 1.f, 1.f, 1.f, 1.f, 1.f, 1.f, 1.f};
#pragma unroll
        for (int i = 0; i < C::FM; ++i) store_rows(i, ones);
    } else {
#pragma unroll
        for (int i = 0; i < C::FM; ++i) {
            float sa[16];
            if (scl) {
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    sa[v] = lsa[r0 + i * 32 + 8 * (v >> 2) + (v & 3)];
            } else {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int dr = i * 32 + 8 * (v >> 2) + (v & 3);
                    sa[v] = dr < rows_left ? j.scale_a[j.m0 + r0 + dr] : 1.0f;
                }
                wait_vmem();
            }
            store_rows(i, sa);
        }
    }
    if (j.wcount) {
        // instrumented launches: one count per stored element
#pragma unroll 1
        for (int i = 0; i < C::FM; ++i)
#pragma unroll 1
            for (int v = 0; v < 16; ++v) {
                const int dr = i * 32 + 8 * (v >> 2) + (v & 3);
                if (dr >= rows_left) continue;
#pragma unroll 1
                for (int jj = 0; jj < C::FN; ++jj)
                    if (jj * 32 < cols_left)
                        atomicAdd(&j.wcount[(int64_t)(j.m0 + r0 + dr) * j.N +
                                            j.n0 + c0 + jj * 32],
                                  1);
            }
    }
}

template <class C>
__device__ __forceinline__ void zero_acc(f32x16 (&acc)[C::FM][C::FN]) {
#pragma unroll
    for (int i = 0; i < C::FM; ++i)
#pragma unroll
        for (int j = 0; j < C::FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
}

// One problem: traversal index -> owned sub-tensor.
template <class C>
struct SingleProvider {
    const GemmArgs &g;
    __device__ int n_prog() const { return g.s.n_prog; }
    __device__ int count() const { return g.s.n_tiles; }
    __device__ Job job(int t) const {
        int tm, tn;
        tile_coords(t, g.s, tm, tn);
        Job j;
        j.a = static_cast<const char *>(g.a);
        j.b = static_cast<const char *>(g.b);
        j.c = g.c;
        // staged programs apply no scales (the host never gives them any),
        // which keeps their epilogue within the register budget
        if constexpr (C::STG) {
            j.scale_a = nullptr; j.scale_b = nullptr;
        } else {
            j.scale_a = g.scale_a; j.scale_b = g.scale_b;
        }
        j.wcount = g.wcount;
        j.lda = g.lda; j.ldb = g.ldb; j.ldc = g.ldc;
        j.M = g.M; j.N = g.N; j.K = g.K;
        j.m0 = tm * C::BM; j.n0 = tn * C::BN;
        set_streams<C>(j);
        return j;
    }
};

// Grouped launch: traversal index -> (problem, owned sub-tensor) by binary
// search on the tile prefix sums of the problem table.
template <class C>
struct GroupProvider {
    const GroupProblem *tab;
    int n, total, G;
    __device__ int n_prog() const { return G; }
    __device__ int count() const { return total; }
    // Sub-tensors stand in the order of falling K and program p takes the
    // p-th of every G.  Every other full row of G is dealt backwards (the
    // last one for certain, so that a partial row after it goes to the
    // programs with least behind them): forwards only, the first programs
    // got the longest of each row and the launch waited for them, 4-6 % at
    // 64 problems, 20-50 % at ten.
    __device__ Job job(int t) const {
        const int row = t / G, rows = total / G;
        if (row < rows && ((rows - 1 - row) & 1) == 0)
            t = row * G + (G - 1 - (t - row * G));
        int lo = 0, hi = n - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (tab[mid].tile_begin <= t) lo = mid; else hi = mid - 1;
        }
        const GroupProblem &pb = tab[lo];
        Sched s;
        s.tiles_m = pb.tiles_m; s.tiles_n = pb.tiles_n;
        s.n_tiles = pb.tiles_m * pb.tiles_n; s.n_prog = G; s.group_m = 8;
        int tm, tn;
        tile_coords(t - pb.tile_begin, s, tm, tn);
        Job j;
        j.a = static_cast<const char *>(pb.a);
        j.b = static_cast<const char *>(pb.b);
        j.c = pb.c;
        j.scale_a = nullptr; j.scale_b = nullptr; j.wcount = pb.wcount;
        j.lda = pb.lda; j.ldb = pb.ldb; j.ldc = pb.ldc;
        j.M = pb.M; j.N = pb.N; j.K = pb.K;
        j.m0 = tm * C::BM; j.n0 = tn * C::BN;
        set_streams<C>(j);
        return j;
    }
};

}  // namespace
}  // namespace tg
