// gemm_tiled.hip -- persistent tile programs for C = A . B on gfx950 MFMA.
//
// One workgroup is one tile program of the mapped-partition schedule
// (Sec. 3.6 of the paper): it owns the output sub-tensors
// program_slot(p) + r*G of the traversal order, and for each of them
//   acc = 0; for every K tile: acc += A[BM x BK] . B[BK x BN]; store acc
// into its own BM x BN sub-tensor only.  A and B are read-only.
//
// gfx950 design:
//   * every K tile is RBY = 128 or 64 bytes deep per row (bf16: 64 or 32
//     elements, e4m3: 128 or 64, f32: 32);
//   * k-contiguous operands (A, and B stored N x K) live in LDS as
//     [rows][128 B] with the 16-byte chunk index XOR-swizzled per row so
//     that the 16-byte fragment reads are free of bank conflicts;
//   * tiles move from HBM to LDS with direct buffer->LDS
//     loads (no staging registers, no LDS write instructions): lane l of a
//     wavefront writes LDS bytes [16 l, 16 l + 16) of a 1 KiB block, so each
//     lane fetches the global chunk that the swizzle assigns to that
//     position; one buffer descriptor per operand and K tile, offsets past
//     its end (rows beyond M or N, K beyond the tail) load zeros;
//   * a bf16 B stored K x N stays k-major in LDS ([BK][BN], chunk index
//     XOR-swizzled by k & 3) and is read with the transposing LDS read,
//     which hands each lane four consecutive k of one column;
//   * a ring of NS = 2 or 4 LDS stages: the loads of the next NS - 1 K tiles
//     are in flight while the MFMAs consume the current one (the HBM/L2
//     latency under full load is about the time of one 64-deep step, so the
//     deeper ring with 32-deep tiles keeps the matrix cores fed); one barrier
//     per K tile; the first K tiles of the program's next sub-tensor are
//     fetched while the current one is stored;
//   * a f32 B stored K x N stays k-major too and is read four bytes at a
//     time, lanes along n (no bank conflicts).  The f32 product is bound by
//     the 32x32x2 instruction (64 cycles each, 157 TFLOP/s nominal); what it
//     lost was waiting: tiles staged through registers at one program per
//     compute unit ran 2048^3 in 171 us and 3072^3 in 815, direct loads 141
//     and 475 (the chip's rate on a large f32 product: 121 and 407).
#include <atomic>
#include <iterator>
#include <vector>

#include "tg_tiled.hpp"

namespace tg {
namespace {

// ---------------------------------------------------------------- compute

// hook(kk, KK) runs once per K step kk (after the step's fragment reads are
// issued for bf16 and f32, before them for e4m3); the direct-load programs
// issue the next K tile's loads from it.
template <class C, class Hook>
__device__ __forceinline__ void compute_stage(const char *stage, int wm,
                                              int wn, int lane,
                                              f32x16 (&acc)[C::FM][C::FN],
                                              Hook hook) {
    const char *As = stage;
    const char *Bs = stage + C::BM * C::RBY;
    const int r = lane & 31, half = lane >> 5;
    // Fragment rows are wm * TM + f * 32 + r (A) and wn * TN + f * 32 + r
    // (B): one lane offset per K step, the rest compile-time constants.
    const int sw = swz_f<C>(r);
    const char *Aw = As + wm * C::TM * C::RBY + r * C::RBY;
    const char *Bw = Bs + wn * C::TN * C::RBY + r * C::RBY;
    if constexpr (C::DTYPE == TG_BF16 || C::DTYPE == TG_F32) {
        // fragments of step kk + 1 are read while the MFMAs of step kk run
        i32x4 af[2][C::FM], bfr[2][C::FN];
        auto load = [&](int kk, int s) {
            const int co = ((2 * kk + half) ^ sw) << 4;
#pragma unroll
            for (int f = 0; f < C::FM; ++f)
                af[s][f] = *reinterpret_cast<const i32x4 *>(
                    Aw + f * 32 * C::RBY + co);
#pragma unroll
            for (int f = 0; f < C::FN; ++f) {
                if constexpr (C::B_KMAJOR && C::DTYPE == TG_F32) {
                    // k = 8 kk + 4 half + e, as the A chunk of this half
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        bfr[s][f][e] = *reinterpret_cast<const int *>(
                            Bs + (8 * kk + 4 * half + e) * C::RB +
                            (wn * C::TN + f * 32 + r) * 4);
                } else if constexpr (C::B_KMAJOR)
                    bfr[s][f] = read_b_kmajor<C>(Bs, kk, wn * C::TN + f * 32,
                                                 lane);
                else
                    bfr[s][f] = *reinterpret_cast<const i32x4 *>(
                        Bw + f * 32 * C::RBY + co);
            }
        };
        constexpr int KK = C::DTYPE == TG_BF16 ? C::BK / 16 : C::BK / 8;
        load(0, 0);
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            const int s = kk & 1;
            if (kk + 1 < KK) load(kk + 1, s ^ 1);
            hook(kk, KK);
            if constexpr (C::DTYPE == TG_BF16 && C::FM * C::FN >= 8) {
                // interleave the next step's LDS reads with this step's
                // MFMAs: one read after each of the first MFMAs
                constexpr int NR = C::FM + (C::B_KMAJOR ? 2 : 1) * C::FN;
                if (kk + 1 < KK) {
#pragma unroll
                    for (int q = 0; q < NR; ++q) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < C::FM; ++i)
#pragma unroll
                for (int j = 0; j < C::FN; ++j) {
                    if constexpr (C::DTYPE == TG_BF16) {
                        acc[i][j] = mfma_bf16(af[s][i], bfr[s][j], acc[i][j]);
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const uint32_t ua = af[s][i][e], ub = bfr[s][j][e];
                            acc[i][j] =
                                mfma_f32(as_f32(ua), as_f32(ub), acc[i][j]);
                        }
                    }
                }
        }
    } else {
#pragma unroll
        for (int kk = 0; kk < C::BK / 64; ++kk) {
            hook(kk, C::BK / 64);   // before this step's fragments are live
            const int c = 4 * kk + 2 * half;
            const int co0 = (c ^ sw) << 4, co1 = ((c + 1) ^ sw) << 4;
            i32x8 af[C::FM], bfr[C::FN];
#pragma unroll
            for (int f = 0; f < C::FM; ++f) {
                i32x4 lo = *reinterpret_cast<const i32x4 *>(Aw + f * 32 * C::RBY + co0);
                i32x4 hi = *reinterpret_cast<const i32x4 *>(Aw + f * 32 * C::RBY + co1);
                af[f] = i32x8{lo[0], lo[1], lo[2], lo[3],
                              hi[0], hi[1], hi[2], hi[3]};
            }
#pragma unroll
            for (int f = 0; f < C::FN; ++f) {
                i32x4 lo = *reinterpret_cast<const i32x4 *>(Bw + f * 32 * C::RBY + co0);
                i32x4 hi = *reinterpret_cast<const i32x4 *>(Bw + f * 32 * C::RBY + co1);
                bfr[f] = i32x8{lo[0], lo[1], lo[2], lo[3],
                               hi[0], hi[1], hi[2], hi[3]};
            }
#pragma unroll
            for (int i = 0; i < C::FM; ++i)
#pragma unroll
                for (int j = 0; j < C::FN; ++j)
                    acc[i][j] = mfma_fp8(af[i], bfr[j], acc[i][j]);
        }
    }
}

// K not a multiple of the 16-byte chunk: the chunk that straddles K was
// loaded as zeros; write its K % EPC valid elements of every row (A, and B
// stored N x K) into LDS one by one.  Called after the stage's loads have
// landed and all wavefronts passed a barrier; a barrier must follow.
template <class C>
__device__ __forceinline__ void fill_k_tail2(const Job &j, char *stage,
                                             char *Bs, int k0, int tid) {
    const int rem = j.K % C::EPC;
    const int kbase = j.K - rem;                  // first element of the chunk
    const int chunk = (kbase - k0) / C::EPC;      // its logical chunk index
    for (int r = tid; r < C::BM; r += C::THREADS) {
        const int row = j.m0 + r;
        char *dst = stage + swz<C>(r, chunk);
        const char *src = j.a + ((int64_t)row * j.lda + kbase) * C::ES;
        for (int e = 0; e < rem; ++e) {
            if constexpr (C::ES == 2)
                reinterpret_cast<uint16_t *>(dst)[e] =
                    row < j.M ? reinterpret_cast<const uint16_t *>(src)[e] : 0;
            else
                reinterpret_cast<uint8_t *>(dst)[e] =
                    row < j.M ? reinterpret_cast<const uint8_t *>(src)[e] : 0;
        }
    }
    if constexpr (!C::B_KMAJOR) {
        for (int r = tid; r < C::BN; r += C::THREADS) {
            const int row = j.n0 + r;
            char *dst = Bs + swz<C>(r, chunk);
            const char *src = j.b + ((int64_t)row * j.ldb + kbase) * C::ES;
            for (int e = 0; e < rem; ++e) {
                if constexpr (C::ES == 2)
                    reinterpret_cast<uint16_t *>(dst)[e] =
                        row < j.N ? reinterpret_cast<const uint16_t *>(src)[e]
                                  : 0;
                else
                    reinterpret_cast<uint8_t *>(dst)[e] =
                        row < j.N ? reinterpret_cast<const uint8_t *>(src)[e]
                                  : 0;
            }
        }
    }
}

template <class C>
__device__ __forceinline__ void fill_k_tail(const Job &j, char *stage, int k0,
                                            int tid) {
    fill_k_tail2<C>(j, stage, stage + C::BM * C::RBY, k0, tid);
}

// ------------------------------------------------------- persistent loops

// Wait until the loads of one K tile have landed while the loads of the
// `later` tiles issued after it (0 <= later <= NS - 2) may still be in
// flight: every wavefront issues the same LPW loads per tile, in tile order.
template <class C>
__device__ __forceinline__ void wait_tile(int later) {
    if constexpr (C::NS >= 4) {
        if (later >= 2) {
            wait_vmem_le<2 * C::LPW>();
            return;
        }
    }
    if constexpr (C::NS >= 3) {
        if (later >= 1) {
            wait_vmem_le<C::LPW>();
            return;
        }
    }
    wait_vmem();
}

// Direct-load programs (bf16, e4m3).  P provides the owned sub-tensors:
// P::n_prog(), P::count(), P::job(t).  The K tiles of all owned sub-tensors
// flow through a ring of NS LDS stages (running index g): tile g lives in
// stage g % NS, and the loads of tiles g+1 .. g+NS-2 are in flight while
// tile g is contracted.
template <class C, class P>
__device__ __forceinline__ void run_direct(const P &prov, char *smem) {
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform
    const int wm = wave / C::WN, wn = wave % C::WN;
    const int G = prov.n_prog(), total = prov.count();
    int t = program_slot(blockIdx.x, G);
    if (t >= total) return;
    auto stage = [&](int g) { return smem + (g % C::NS) * C::STAGE; };
    auto slot = [&](int n) { return scale_slot<C>(smem, n); };
    Job j = prov.job(t);
    int g = 0, njob = 0;
    {
        const int nk = (j.K + C::BK - 1) / C::BK;
        issue_scales<C>(j, slot(njob), wave, lane);
        for (int s = 0; s < C::NS - 1 && s < nk; ++s)
            issue_direct<C>(j, stage(g + s), s * C::BK, wave, lane);
    }
    f32x16 acc[C::FM][C::FN];
    while (true) {
        const int nk = (j.K + C::BK - 1) / C::BK;
        // the last K tile holds a chunk that straddles K
        const bool ragged = (j.K % C::EPC) != 0;
        zero_acc<C>(acc);
        if (nk == 0) {
            wait_vmem();      // the scales
            ring_barrier();
        }
        for (int kt = 0; kt < nk; ++kt) {
            const int later = nk - 1 - kt < C::NS - 2 ? nk - 1 - kt : C::NS - 2;
            if (kt == 0)
                wait_vmem();   // also covers the previous sub-tensor's stores
            else
                wait_tile<C>(later);
            ring_barrier();
            if (ragged && kt == nk - 1) {
                fill_k_tail<C>(j, stage(g + kt), kt * C::BK, tid);
                __syncthreads();
            }
            // the stage of tile kt - 1 is free: every wavefront passed the
            // barrier above after contracting it.  The loads of tile
            // kt + NS - 1 are issued inside the contraction, the A tile
            // after the first K step's fragment reads and the B tile one
            // step later, so the MFMA pipe is fed while they issue.
            const bool nxt = kt + C::NS - 1 < nk;
            compute_stage<C>(stage(g + kt), wm, wn, lane, acc,
                             [&](int kk, int KK) {
                if (!nxt) return;
                // e4m3 K steps are twice as long: both at the first
                const int parts =
                    C::DTYPE == TG_FP8_E4M3
                        ? (kk == 0 ? 3 : 0)
                        : (kk == 0 ? 1 : 0) | (kk == (KK > 1 ? 1 : 0) ? 2 : 0);
                if (parts)
                    issue_direct<C>(j, stage(g + kt + C::NS - 1),
                                    (kt + C::NS - 1) * C::BK, wave, lane,
                                    parts);
            });
        }
        g += nk;
        // first tiles of the next owned sub-tensor, then store this one; the
        // stages written now are all but the one of the last tile contracted
        t += G;
        const bool more = t < total;
        Job nj;
        if (more) {
            nj = prov.job(t);
            const int nk2 = (nj.K + C::BK - 1) / C::BK;
            issue_scales<C>(nj, slot(njob + 1), wave, lane);
            for (int s = 0; s < C::NS - 1 && s < nk2; ++s)
                issue_direct<C>(nj, stage(g + s), s * C::BK, wave, lane);
        }
        epilogue<C>(j, wm, wn, lane, acc, slot(njob));
        if (!more) break;
        j = nj;
        ++njob;
    }
}

// bf16 fragments of K step kk of a stage: FM A fragments (rows
// wm * TM + f * 32 + lane % 32) and FN B fragments, eight k each.
template <class C>
__device__ __forceinline__ void read_frags2(const char *As, const char *Bs,
                                            int wm, int wn, int lane, int kk,
                                            i32x4 (&af)[C::FM],
                                            i32x4 (&bf)[C::FN]) {
    const int r = lane & 31, half = lane >> 5;
    const int co = ((2 * kk + half) ^ swz_f<C>(r)) << 4;
    const char *Aw = As + wm * C::TM * C::RBY + r * C::RBY + co;
#pragma unroll
    for (int f = 0; f < C::FM; ++f)
        af[f] = *reinterpret_cast<const i32x4 *>(Aw + f * 32 * C::RBY);
#pragma unroll
    for (int f = 0; f < C::FN; ++f) {
        if constexpr (C::B_KMAJOR)
            bf[f] = read_b_kmajor<C>(Bs, kk, wn * C::TN + f * 32, lane);
        else
            bf[f] = *reinterpret_cast<const i32x4 *>(
                Bs + (wn * C::TN + f * 32 + r) * C::RBY + co);
    }
}

template <class C>
__device__ __forceinline__ void read_frags(const char *stage, int wm, int wn,
                                           int lane, int kk,
                                           i32x4 (&af)[C::FM],
                                           i32x4 (&bf)[C::FN]) {
    read_frags2<C>(stage, stage + C::BM * C::RBY, wm, wn, lane, kk, af, bf);
}

// The MFMAs of one K step, with the fragment reads issued just before
// them interleaved one by one (NR of them).
template <class C, int NR>
__device__ __forceinline__ void mfma_step(const i32x4 (&af)[C::FM],
                                          const i32x4 (&bf)[C::FN],
                                          f32x16 (&acc)[C::FM][C::FN]) {
#pragma unroll
    for (int q = 0; q < NR; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
#pragma unroll
    for (int i = 0; i < C::FM; ++i)
#pragma unroll
        for (int jj = 0; jj < C::FN; ++jj)
            acc[i][jj] = mfma_bf16(af[i], bf[jj], acc[i][jj]);
}


// Cross-tile schedule (bf16).  The barrier that hands over K tile kt + 1
// sits before the last K step of tile kt instead of after it: every
// wavefront has read all of tile kt's fragments by then, so the stage of
// tile kt is free for the loads of tile kt + NS, and the first fragments
// of tile kt + 1 are read while the last MFMAs of tile kt run.  The wait
// for the barrier and the LDS latency of the next tile's first reads are
// thereby covered by MFMA work.  Same ring and load accounting as the
// lock-step loop: tile g in stage g % NS, every wavefront issues LPW loads
// per tile in tile order.
template <class C, class P>
__device__ __forceinline__ void run_direct_xt(const P &prov, char *smem) {
    constexpr int KK = C::BK / 16;                 // K steps per tile (even)
    constexpr int NR = C::FM + (C::B_KMAJOR ? 2 : 1) * C::FN;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform
    const int wm = wave / C::WN, wn = wave % C::WN;
    const int G = prov.n_prog(), total = prov.count();
    int t = program_slot(blockIdx.x, G);
    if (t >= total) return;
    auto stage = [&](int g) { return smem + (g % C::NS) * C::STAGE; };
    Job j = prov.job(t);
    int g = 0;
    {
        const int nk = (j.K + C::BK - 1) / C::BK;
        for (int s = 0; s < C::NS - 1 && s < nk; ++s)
            issue_direct<C>(j, stage(g + s), s * C::BK, wave, lane);
    }
    f32x16 acc[C::FM][C::FN];
    i32x4 fa[2][C::FM], fb[2][C::FN];
    while (true) {
        const int nk = (j.K + C::BK - 1) / C::BK;
        const bool ragged = (j.K % C::EPC) != 0;
        zero_acc<C>(acc);
        wait_vmem();          // also covers the previous sub-tensor's stores
        ring_barrier();
        if (nk > 0) {
            if (ragged && nk == 1) {
                fill_k_tail<C>(j, stage(g), 0, tid);
                __syncthreads();
            }
            // the stage of the previous sub-tensor's last tile is free
            if (C::NS - 1 < nk)
                issue_direct<C>(j, stage(g + C::NS - 1),
                                (C::NS - 1) * C::BK, wave, lane);
            read_frags<C>(stage(g), wm, wn, lane, 0, fa[0], fb[0]);
        }
        int pend_b = -1;      // tile whose B loads are still to be issued
        for (int kt = 0; kt < nk; ++kt) {
            char *st = stage(g + kt);
#pragma unroll
            for (int kk = 0; kk < KK - 1; ++kk) {
                const int s = kk & 1;
                read_frags<C>(st, wm, wn, lane, kk + 1, fa[s ^ 1], fb[s ^ 1]);
                mfma_step<C, NR>(fa[s], fb[s], acc);
                if (kk == 0 && pend_b >= 0) {
                    issue_direct<C>(j, stage(g + pend_b), pend_b * C::BK,
                                    wave, lane, 2);
                    pend_b = -1;
                }
            }
            // tile kt + 1 has landed for every wavefront and nobody reads
            // tile kt any more.  After the last tile the barrier and the
            // reads of the (unused) next stage still run, keeping the loop
            // free of a second copy of the MFMAs.
            const int later = nk - 2 - kt < C::NS - 2 ? nk - 2 - kt
                                                      : C::NS - 2;
            // (pinned: the scheduler would otherwise hoist the barrier
            // above the MFMAs of the previous steps)
            __builtin_amdgcn_sched_barrier(0);
            wait_tile<C>(later);
            ring_barrier();
            __builtin_amdgcn_sched_barrier(0);
            if (ragged && kt + 1 == nk - 1) {
                fill_k_tail<C>(j, stage(g + kt + 1), (kt + 1) * C::BK, tid);
                __syncthreads();
            }
            read_frags<C>(stage(g + kt + 1), wm, wn, lane, 0, fa[0], fb[0]);
            mfma_step<C, NR>(fa[1], fb[1], acc);
            if (kt + C::NS < nk) {
                issue_direct<C>(j, st, (kt + C::NS) * C::BK, wave, lane, 1);
                pend_b = kt + C::NS;
            }
        }
        g += nk;
        // first tiles of the next owned sub-tensor into every stage but the
        // one of the last tile contracted, then store this one
        t += G;
        const bool more = t < total;
        Job nj;
        if (more) {
            nj = prov.job(t);
            const int nk2 = (nj.K + C::BK - 1) / C::BK;
            for (int s = 0; s < C::NS - 1 && s < nk2; ++s)
                issue_direct<C>(nj, stage(g + s), s * C::BK, wave, lane);
        }
        epilogue<C>(j, wm, wn, lane, acc, nullptr);
        if (!more) break;
        j = nj;
    }
}

// Cross-tile schedule over a ring of five 32-deep slots (bf16, 64-byte K
// rows; five slots fill the 160 KiB of LDS).  The hand-over barrier comes
// every second slot (a 64-deep unit, four K steps), before the unit's last
// K step as in run_direct_xt.  At a hand-over the two slots of the next
// unit have landed and the slot after them may still be in flight, so half
// of the loads of every unit have two unit periods to land and only the
// other half has one.  Slot q of a sub-tensor (running index g + q) lives
// at position (g + q) % 5; a sub-tensor with an odd number of slots gets
// one more, past K, which loads as zeros.  Per wavefront, slot q is issued
// as one group of LPW loads: slots 0 .. 2 before the sub-tensor's first
// barrier (with the previous sub-tensor's store), slot 2u + 3 after the
// last K step of unit u - 1 and slot 2u + 4 after the first K step of unit
// u, so that the hand-over of unit u waits for all but slot 2u + 4.
template <class C, class P>
__device__ __forceinline__ void run_direct_x5(const P &prov, char *smem) {
    static_assert(C::NS == 5 && C::BK == 32, "five slots of 32 K");
    constexpr int NR = C::FM + (C::B_KMAJOR ? 2 : 1) * C::FN;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform
    const int wm = wave / C::WN, wn = wave % C::WN;
    const int G = prov.n_prog(), total = prov.count();
    int t = program_slot(blockIdx.x, G);
    if (t >= total) return;
    auto slot = [&](int q) { return smem + (q % 5) * C::STAGE; };
    auto nslots = [&](const Job &jb) {
        return (((jb.K + C::BK - 1) / C::BK) + 1) & ~1;
    };
    Job j = prov.job(t);
    int g = 0;
    {
        const int nq = nslots(j);
        for (int q = 0; q < 3 && q < nq; ++q)
            issue_direct<C>(j, slot(g + q), q * C::BK, wave, lane);
    }
    f32x16 acc[C::FM][C::FN];
    i32x4 fa[2][C::FM], fb[2][C::FN];
    while (true) {
        const int nq = nslots(j), nu = nq / 2;
        const bool ragged = (j.K % C::EPC) != 0;
        const int qtail = (j.K + C::BK - 1) / C::BK - 1;  // straddling chunk
        zero_acc<C>(acc);
        wait_vmem();          // also covers the previous sub-tensor's stores
        ring_barrier();
        int pend = -1;        // slot to issue after the next first K step
        if (nu > 0) {
            if (ragged && qtail <= 1) {
                fill_k_tail<C>(j, slot(g + qtail), qtail * C::BK, tid);
                __syncthreads();
            }
            if (3 < nq) issue_direct<C>(j, slot(g + 3), 3 * C::BK, wave, lane);
            if (4 < nq) pend = 4;
            read_frags<C>(slot(g), wm, wn, lane, 0, fa[0], fb[0]);
        }
        for (int u = 0; u < nu; ++u) {
            char *sa = slot(g + 2 * u), *sb = slot(g + 2 * u + 1);
            read_frags<C>(sa, wm, wn, lane, 1, fa[1], fb[1]);
            mfma_step<C, NR>(fa[0], fb[0], acc);
            if (pend >= 0) {
                issue_direct<C>(j, slot(g + pend), pend * C::BK, wave, lane);
                pend = -1;
            }
            read_frags<C>(sb, wm, wn, lane, 0, fa[0], fb[0]);
            mfma_step<C, NR>(fa[1], fb[1], acc);
            read_frags<C>(sb, wm, wn, lane, 1, fa[1], fb[1]);
            mfma_step<C, NR>(fa[0], fb[0], acc);
            // hand-over of unit u + 1 (pinned, as in run_direct_xt); after
            // the last unit it still runs and reads an unused slot
            __builtin_amdgcn_sched_barrier(0);
            if (2 * u + 4 < nq)
                wait_vmem_le<C::LPW>();
            else
                wait_vmem();
            ring_barrier();
            __builtin_amdgcn_sched_barrier(0);
            if (ragged && (qtail >> 1) == u + 1) {
                fill_k_tail<C>(j, slot(g + qtail), qtail * C::BK, tid);
                __syncthreads();
            }
            read_frags<C>(slot(g + 2 * u + 2), wm, wn, lane, 0, fa[0], fb[0]);
            mfma_step<C, NR>(fa[1], fb[1], acc);
            // the positions of unit u are free now
            if (2 * u + 5 < nq)
                issue_direct<C>(j, sa, (2 * u + 5) * C::BK, wave, lane);
            if (2 * u + 6 < nq) pend = 2 * u + 6;
        }
        g += nq;
        // slots 0 .. 2 of the next owned sub-tensor go to the three
        // positions other than those of the last unit, then this one is
        // stored
        t += G;
        const bool more = t < total;
        Job nj;
        if (more) {
            nj = prov.job(t);
            const int nq2 = nslots(nj);
            for (int q = 0; q < 3 && q < nq2; ++q)
                issue_direct<C>(nj, slot(g + q), q * C::BK, wave, lane);
        }
        epilogue<C>(j, wm, wn, lane, acc, nullptr);
        if (!more) break;
        j = nj;
    }
}

// Cross-tile schedule over five operand slots (bf16, 64-deep K tiles,
// BM = BN): each slot holds the A or the B tile of one K tile, so the
// 160 KiB of LDS hold two and a half K tiles.  Operand q of a sub-tensor
// (A of tile t is q = 2t, B is q = 2t + 1; running index g + q) lives in
// slot (g + q) % 5.  At the hand-over of tile kt + 1 (before the last K
// step of tile kt) the slots of tile kt are freed: the B tile of kt + 2
// goes into one right away and the A tile of kt + 3 into the other after
// the next tile's first K step, so that A tiles are in flight for about
// two tile periods and B tiles for about one (two-stage ring: one and a
// bit less).  The hand-over waits for tile kt + 1 while the A tile of
// kt + 2, issued last, may still be in flight.
template <class C, class P>
__device__ __forceinline__ void run_direct_xh(const P &prov, char *smem) {
    static_assert(C::HALVES && C::BM == C::BN, "five operand slots");
    constexpr int KK = C::BK / 16;
    constexpr int NR = C::FM + (C::B_KMAJOR ? 2 : 1) * C::FN;
    constexpr int HALF = C::STAGE / 2;
    constexpr int LPA = C::BM * C::RBY / 1024 / C::NW;  // loads per A tile
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform
    const int wm = wave / C::WN, wn = wave % C::WN;
    const int G = prov.n_prog(), total = prov.count();
    int t = program_slot(blockIdx.x, G);
    if (t >= total) return;
    auto slot = [&](int q) { return smem + (q % 5) * HALF; };
    Job j = prov.job(t);
    int g = 0;
    {
        const int nk = (j.K + C::BK - 1) / C::BK;
        if (nk > 0) {
            issue_a<C>(j, slot(g), 0, wave, lane);
            issue_b<C>(j, slot(g + 1), 0, wave, lane);
        }
        if (nk > 1) issue_a<C>(j, slot(g + 2), C::BK, wave, lane);
    }
    f32x16 acc[C::FM][C::FN];
    i32x4 fa[2][C::FM], fb[2][C::FN];
    while (true) {
        const int nk = (j.K + C::BK - 1) / C::BK;
        const bool ragged = (j.K % C::EPC) != 0;
        zero_acc<C>(acc);
        wait_vmem();          // also covers the previous sub-tensor's stores
        ring_barrier();
        if (nk > 0) {
            if (ragged && nk == 1) {
                fill_k_tail2<C>(j, slot(g), slot(g + 1), 0, tid);
                __syncthreads();
            }
            // the slots of the previous sub-tensor's last tile are free
            if (nk > 1) issue_b<C>(j, slot(g + 3), C::BK, wave, lane);
            read_frags2<C>(slot(g), slot(g + 1), wm, wn, lane, 0, fa[0],
                           fb[0]);
        }
        for (int kt = 0; kt < nk; ++kt) {
            const char *sa = slot(g + 2 * kt), *sb = slot(g + 2 * kt + 1);
#pragma unroll
            for (int kk = 0; kk < KK - 1; ++kk) {
                const int s = kk & 1;
                read_frags2<C>(sa, sb, wm, wn, lane, kk + 1, fa[s ^ 1],
                               fb[s ^ 1]);
                mfma_step<C, NR>(fa[s], fb[s], acc);
                if (kk == 0 && kt + 2 < nk)   // into the slot of B of kt - 1
                    issue_a<C>(j, slot(g + 2 * kt + 4), (kt + 2) * C::BK,
                               wave, lane);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (kt + 2 < nk)
                wait_vmem_le<LPA>();
            else
                wait_vmem();
            ring_barrier();
            __builtin_amdgcn_sched_barrier(0);
            if (ragged && kt + 1 == nk - 1) {
                fill_k_tail2<C>(j, slot(g + 2 * kt + 2), slot(g + 2 * kt + 3),
                                (kt + 1) * C::BK, tid);
                __syncthreads();
            }
            read_frags2<C>(slot(g + 2 * kt + 2), slot(g + 2 * kt + 3), wm, wn,
                           lane, 0, fa[0], fb[0]);
            mfma_step<C, NR>(fa[1], fb[1], acc);
            if (kt + 2 < nk)                  // into the slot of A of kt
                issue_b<C>(j, slot(g + 2 * kt + 5), (kt + 2) * C::BK, wave,
                           lane);
        }
        g += 2 * nk;
        // A and B of the next sub-tensor's first tile and its second A go
        // to the three slots other than those of the last tile, then this
        // one is stored
        t += G;
        const bool more = t < total;
        Job nj;
        if (more) {
            nj = prov.job(t);
            const int nk2 = (nj.K + C::BK - 1) / C::BK;
            if (nk2 > 0) {
                issue_a<C>(nj, slot(g), 0, wave, lane);
                issue_b<C>(nj, slot(g + 1), 0, wave, lane);
            }
            if (nk2 > 1) issue_a<C>(nj, slot(g + 2), C::BK, wave, lane);
        }
        epilogue<C>(j, wm, wn, lane, acc, nullptr);
        if (!more) break;
        j = nj;
    }
}


// ------------------------------------------------------ ping-pong schedule
//
// Eight wavefronts in two groups of four (group = wm); the hardware places
// wavefront w on SIMD w % 4, so every SIMD holds one wavefront of each
// group.  The groups run the same sequence of phases, one phase apart:
//   MEM(q):  issue the HBM -> LDS loads of K tile q + NS - 1, then read this
//            wavefront's fragments of K tile q from LDS into registers;
//   COMP(q): the MFMAs of K tile q, from registers only.
// A workgroup barrier separates consecutive phases, so while one group
// contracts, the other group's LDS reads and load issue run on the same
// SIMDs, and the MFMA pipe of each SIMD is fed from one long run of
// independent instructions.  K tiles of consecutive owned sub-tensors form
// one stream q = 0, 1, ...; the loads run NS - 1 tiles ahead.
//
// Ordering (phase k starts at barrier k; group 0 runs MEM(q) in phase 2q
// and COMP(q) in 2q + 1, group 1 one phase later):
//  * tile q is first read in phase 2q: every wavefront waits for its own
//    loads of tile q before barrier 2q (group 0 before MEM(q), group 1
//    before COMP(q - 1));
//  * the loads of tile q + NS - 1 overwrite the stage of tile q - 1, whose
//    last reader (group 1, MEM(q - 1), phase 2q - 1) finished its LDS reads
//    before barrier 2q, the earliest issue of those loads;
//  * both groups pass the same number of barriers: group 1 one extra at the
//    start, group 0 one extra at the end.
template <class C>
struct PPFrag {
    static constexpr bool F8 = C::DTYPE == TG_FP8_E4M3;
    static constexpr int KS = F8 ? C::BK / 64 : C::BK / 16;  // MFMA K steps
    static constexpr int W = F8 ? 2 : 1;                     // i32x4 / operand
    i32x4 a[KS][C::FM][W];
    i32x4 b[KS][C::FN][W];
};

template <class C>
__device__ __forceinline__ void pp_read(const char *stage, int wm, int wn,
                                        int lane, PPFrag<C> &f) {
    const char *As = stage;
    const char *Bs = stage + C::BM * C::RBY;
    const int r = lane & 31, half = lane >> 5;
#pragma unroll
    for (int ks = 0; ks < PPFrag<C>::KS; ++ks) {
        const int c = PPFrag<C>::F8 ? 4 * ks + 2 * half : 2 * ks + half;
#pragma unroll
        for (int i = 0; i < C::FM; ++i)
#pragma unroll
            for (int w = 0; w < PPFrag<C>::W; ++w)
                f.a[ks][i][w] = *reinterpret_cast<const i32x4 *>(
                    As + swz<C>(wm * C::TM + i * 32 + r, c + w));
#pragma unroll
        for (int jj = 0; jj < C::FN; ++jj) {
            if constexpr (C::B_KMAJOR) {
                f.b[ks][jj][0] =
                    read_b_kmajor<C>(Bs, ks, wn * C::TN + jj * 32, lane);
            } else {
#pragma unroll
                for (int w = 0; w < PPFrag<C>::W; ++w)
                    f.b[ks][jj][w] = *reinterpret_cast<const i32x4 *>(
                        Bs + swz<C>(wn * C::TN + jj * 32 + r, c + w));
            }
        }
    }
}

template <class C>
__device__ __forceinline__ void pp_mfma(const PPFrag<C> &f,
                                        f32x16 (&acc)[C::FM][C::FN]) {
#pragma unroll
    for (int ks = 0; ks < PPFrag<C>::KS; ++ks)
#pragma unroll
        for (int i = 0; i < C::FM; ++i)
#pragma unroll
            for (int jj = 0; jj < C::FN; ++jj) {
                if constexpr (PPFrag<C>::F8) {
                    const i32x4 a0 = f.a[ks][i][0], a1 = f.a[ks][i][1];
                    const i32x4 b0 = f.b[ks][jj][0], b1 = f.b[ks][jj][1];
                    acc[i][jj] = mfma_fp8(
                        i32x8{a0[0], a0[1], a0[2], a0[3], a1[0], a1[1], a1[2],
                              a1[3]},
                        i32x8{b0[0], b0[1], b0[2], b0[3], b1[0], b1[1], b1[2],
                              b1[3]},
                        acc[i][jj]);
                } else {
                    acc[i][jj] = mfma_bf16(f.a[ks][i][0], f.b[ks][jj][0],
                                           acc[i][jj]);
                }
            }
}

// Barrier between two phases: this wavefront's LDS reads are complete, and
// no instruction moves across it.
__device__ __forceinline__ void phase_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    ring_barrier();
    __builtin_amdgcn_sched_barrier(0);
}

// K tiles of one owned sub-tensor in the stream; K = 0 takes one tile of
// zeros (every chunk lies beyond K and loads as zeros).
template <class C>
__device__ __forceinline__ int pp_tiles(int K) {
    const int nk = (K + C::BK - 1) / C::BK;
    return nk > 0 ? nk : 1;
}

// Loads of the K-tile stream in issue order: (owned sub-tensor, K tile).
// A sub-tensor's scales are issued with its first K tile, into the LDS
// slot of its position in the sequence of owned sub-tensors.
template <class C, class P>
struct LoadCursor {
    const P &prov;
    Job j;
    int t, kt, nk, total, G;
    int issued;   // tiles issued so far (stream index of the next one)
    int njob;     // position of j among this program's sub-tensors

    __device__ LoadCursor(const P &p, int t0, int total_, int G_)
        : prov(p), t(t0), kt(0), total(total_), G(G_), issued(0), njob(0) {
        j = prov.job(t);
        nk = pp_tiles<C>(j.K);
    }
    __device__ __forceinline__ void issue(char *smem, int wave, int lane) {
        if (t >= total) return;
        if (kt == 0)
            issue_scales<C>(j, scale_slot<C>(smem, njob), wave, lane);
        issue_direct<C>(j, smem + (issued % C::NS) * C::STAGE, kt * C::BK,
                        wave, lane);
        ++issued;
        if (++kt == nk) {
            kt = 0;
            t += G;
            ++njob;
            if (t < total) {
                j = prov.job(t);
                nk = pp_tiles<C>(j.K);
            }
        }
    }
};

// Wait until this wavefront's loads of stream tile q have landed.  Loads
// complete in issue order; after epilogue stores (dirty) everything is
// drained, since stores need not complete in order with loads.
template <class C>
__device__ __forceinline__ void pp_wait(int q, int issued, bool &dirty) {
    if (q >= issued) return;   // past the end of the stream
    if (dirty) {
        wait_vmem();
        dirty = false;
        return;
    }
    int later = issued - 1 - q;
    later = later < C::NS - 2 ? later : C::NS - 2;
    wait_tile<C>(later);
}

// Ping-pong programs (bf16, e4m3; K a positive multiple of the 16-byte
// chunk, so no tile needs a tail fill).
template <class C, class P>
__device__ __forceinline__ void run_pingpong(const P &prov, char *smem) {
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform
    const int wm = wave / C::WN, wn = wave % C::WN;
    const int grp = wm;
    const int G = prov.n_prog(), total = prov.count();
    int t = program_slot(blockIdx.x, G);
    if (t >= total) return;
    LoadCursor<C, P> ld(prov, t, total, G);
    for (int s = 0; s < C::NS - 1; ++s) ld.issue(smem, wave, lane);
    Job j = prov.job(t);
    int nk = pp_tiles<C>(j.K);
    int kt = 0, q = 0, njob = 0;
    bool dirty = false;
    f32x16 acc[C::FM][C::FN];
    zero_acc<C>(acc);
    PPFrag<C> f;
    if (grp == 1) {
        pp_wait<C>(0, ld.issued, dirty);
        phase_barrier();
    }
    while (true) {
        // MEM(q)
        if (grp == 0) pp_wait<C>(q, ld.issued, dirty);
        phase_barrier();
        ld.issue(smem, wave, lane);
        pp_read<C>(smem + (q % C::NS) * C::STAGE, wm, wn, lane, f);
        // COMP(q)
        if (grp == 1) pp_wait<C>(q + 1, ld.issued, dirty);
        phase_barrier();
        __builtin_amdgcn_s_setprio(1);
        pp_mfma<C>(f, acc);
        __builtin_amdgcn_s_setprio(0);
        ++q;
        if (++kt == nk) {
            epilogue<C>(j, wm, wn, lane, acc, scale_slot<C>(smem, njob));
            ++njob;
            dirty = true;
            t += G;
            if (t >= total) break;
            j = prov.job(t);
            nk = pp_tiles<C>(j.K);
            kt = 0;
            zero_acc<C>(acc);
        }
    }
    if (grp == 0) phase_barrier();
}


// ------------------------------------------------------- bulk-read ring
//
// Bulk-read schedule (bf16, A and B both k-contiguous).  A K tile's
// fragments are read from LDS into registers all at once, one tile period
// before they are contracted, so its LDS stage is free again as soon as
// every wavefront has read it: with a ring of NS stages the direct loads
// of a tile are issued NS - 1 tile periods before the tile is read (the
// lead time that the HBM and L2 latency under full load asks for), and
// each wavefront holds two tiles of fragments (the one being contracted
// and the next).  Four wavefronts of 128 x 128 outputs, one per SIMD,
// accumulators in the AGPR half of the register file.
//
// The loads run as one stream over the K tiles of all owned sub-tensors
// (tile q of the stream in stage q % NS).  Iteration q, with tile q's
// fragments in registers:
//   wait: this wavefront's reads of tile q are complete and its loads of
//         tile q + 1 have landed; barrier (so for every wavefront);
//   issue the loads of tile q + NS into stage q % NS (tile q's, now free);
//   read tile q + 1's fragments into the other register set, one read
//   slotted after each of the first MFMAs of tile q;
//   after the sub-tensor's last tile, store it and start the next.
// Loads complete in issue order, so waiting until at most the loads of the
// tiles issued after tile q + 1 are outstanding means tile q + 1 has
// landed; epilogue stores in between only make that wait longer.

// One 16-byte-per-lane load into LDS at `lds` + 16 * lane from buffer
// `srd` at byte offset voff + soff (same protocol as dma16; the scalar
// offset carries the distance between a wavefront's 1 KiB blocks).
template <bool FIRST>
__device__ __forceinline__ void dma16_so(const i32x4 &srd, uint32_t lds_,
                                         uint32_t voff, int soff) {
    const uint32_t lds = __builtin_amdgcn_readfirstlane(lds_);
    if constexpr (FIRST)
        asm volatile(
            "s_nop 4\n\ts_mov_b32 m0, %0\n\ts_nop 0\n\t"
            "buffer_load_dwordx4 %1, %2, %3 offen lds"
            :
            : "s"(lds), "v"(voff), "s"(srd), "s"(soff)
            : "memory", "m0");
    else
        asm volatile(
            "s_mov_b32 m0, %0\n\ts_nop 0\n\t"
            "buffer_load_dwordx4 %1, %2, %3 offen lds"
            :
            : "s"(lds), "v"(voff), "s"(srd), "s"(soff)
            : "memory", "m0");
}

// Load stream of one operand of one owned sub-tensor (rows k-contiguous):
// first byte of its rows and the bytes from there to the operand's end,
// the lane's offset within the wavefront's first 1 KiB block (block i of
// the wavefront holds rows i * NW * RPK further down; the swizzle repeats
// every 32 rows, so every block of a lane reads the same logical chunk)
// and the distance between blocks.  K is a whole number of K tiles, so no
// chunk straddles or passes K; rows beyond M / N lie past the buffer's
// end and load zeros.
struct BulkStream {
    const char *row;
    int64_t rem;
    uint32_t voff;
    int32_t stride;
};

template <class C>
__device__ __forceinline__ BulkStream bulk_stream(const char *row0,
                                                  int64_t rem, int64_t ld,
                                                  int wave, int lane) {
    static_assert((C::NW * C::RPK) % 32 == 0, "swizzle period");
    BulkStream s;
    const int row = wave * C::RPK + lane / C::CPRW;
    const int kc = (lane % C::CPRW) ^ swz_f<C>(row);
    s.row = row0;
    s.rem = rem;
    s.voff = (uint32_t)((row * ld + kc * C::EPC) * C::ES);
    s.stride = __builtin_amdgcn_readfirstlane(
        (int)(C::NW * C::RPK * ld * C::ES));
    return s;
}

// This wavefront's ROWS / RPK / NW blocks of one operand of K tile k0.
template <class C, int ROWS>
__device__ __forceinline__ void bulk_issue(const BulkStream &s, int k0,
                                           uint32_t dst, int wave) {
    const int64_t skip = (int64_t)k0 * C::ES;
    const i32x4 srd = make_srd(s.row + skip, sat_bytes(s.rem - skip));
#pragma unroll
    for (int i = 0; i < ROWS / C::RPK / C::NW; ++i) {
        const uint32_t lds = dst + (uint32_t)((i * C::NW + wave) * 1024);
        if (i == 0)
            dma16_so<true>(srd, lds, s.voff, 0);
        else
            dma16_so<false>(srd, lds, s.voff,
                            __builtin_amdgcn_readfirstlane(i * s.stride));
    }
}

// The next K tile of the load stream, ready to issue: buffer resources
// of its A and B rows from its first K column and its LDS stage.
struct BulkTile {
    i32x4 sa, sb;
    uint32_t lds;
    bool live;   // the stream has this tile
};

// Loads of the stream in issue order (owned sub-tensor, K tile).
template <class C, class P>
struct BulkCursor {
    const P &prov;
    BulkStream sa, sb;
    int t, kt, nk, total, G;
    int issued;   // tiles issued so far
    int wave, lane;

    __device__ __forceinline__ void start(int t0) {
        const Job j = prov.job(t0);
        nk = pp_tiles<C>(j.K);
        // K = 0 takes one tile of zeros: an empty buffer range
        const bool k0 = j.K == 0;
        sa = bulk_stream<C>(j.a_row, k0 ? 0 : j.a_rem, j.lda, wave, lane);
        sb = bulk_stream<C>(j.b_row, k0 ? 0 : j.b_rem, j.ldb, wave, lane);
    }
    __device__ BulkCursor(const P &p, int t0, int total_, int G_, int w,
                          int l)
        : prov(p), t(t0), kt(0), total(total_), G(G_), issued(0), wave(w),
          lane(l) {
        start(t0);
    }
    __device__ __forceinline__ BulkTile prepare(char *smem) const {
        BulkTile T;
        T.live = t < total;
        const int64_t skip = (int64_t)kt * C::BK * C::ES;
        T.sa = make_srd(sa.row + skip, sat_bytes(sa.rem - skip));
        T.sb = make_srd(sb.row + skip, sat_bytes(sb.rem - skip));
        T.lds = lds_addr(smem) + (uint32_t)((issued % C::NS) * C::STAGE);
        return T;
    }
    // load r of this wavefront's share of the tile: A blocks first, then B
    __device__ __forceinline__ void load(const BulkTile &T, int r) const {
        constexpr int NA = C::BM / C::RPK / C::NW;
        const bool a = r < NA;
        const int i = a ? r : r - NA;
        const uint32_t lds = T.lds + (a ? 0u : (uint32_t)(C::BM * C::RBY)) +
                             (uint32_t)((i * C::NW + wave) * 1024);
        const BulkStream &st = a ? sa : sb;
        if (i == 0)
            dma16_so<true>(a ? T.sa : T.sb, lds, st.voff, 0);
        else
            dma16_so<false>(a ? T.sa : T.sb, lds, st.voff,
                            __builtin_amdgcn_readfirstlane(i * st.stride));
    }
    __device__ __forceinline__ void advance() {
        ++issued;
        if (++kt == nk) {
            kt = 0;
            t += G;
            if (t < total) start(t);
        }
    }
    __device__ __forceinline__ void issue(char *smem) {
        const BulkTile T = prepare(smem);
        if (!T.live) return;
#pragma unroll
        for (int r = 0; r < C::LPW; ++r) load(T, r);
        advance();
    }
};

template <class C>
struct BulkFrags {
    i32x4 a[C::BK / 16][C::FM];
    i32x4 b[C::BK / 16][C::FN];
};

// Wait until at most the loads of `later` tiles (0 <= later < NS) are
// outstanding.
template <class C>
__device__ __forceinline__ void wait_later(int later) {
    static_assert(C::NS <= 5, "wait table");
    switch (later) {
    case 0: wait_vmem(); break;
    case 1: wait_vmem_le<C::LPW>(); break;
    case 2: wait_vmem_le<2 * C::LPW>(); break;
    case 3: wait_vmem_le<3 * C::LPW>(); break;
    default: wait_vmem_le<(C::NS - 1) * C::LPW>(); break;
    }
}

// Barrier of the bulk-read ring: this wavefront's LDS reads are complete
// (a wait the compiler sees, so that it knows the fragments read before
// are in registers and inserts no waits of its own for them), then the
// workgroup barrier.
__device__ __forceinline__ void bulk_barrier() {
    // lgkmcnt(0); vmcnt and expcnt at their no-wait maxima
    __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4));
    __builtin_amdgcn_s_barrier();
}

// One iteration of the bulk-read ring: contract tile q (fragments in cur)
// and read tile q + 1 into nxt.  The tile's MFMAs are cut into LPW groups;
// one load of tile q + NS leads each group (with one wavefront per SIMD a
// load that waits to issue stalls the MFMAs behind it, so the loads are
// spread over the whole tile period), and the fragment reads of tile
// q + 1 are slotted one after each MFMA of the first groups.
template <class C, class P>
__device__ __forceinline__ void bulk_iter(BulkCursor<C, P> &ld, char *smem,
                                          int q, int wave, int lane, int wm,
                                          int wn, const BulkFrags<C> &cur,
                                          BulkFrags<C> &nxt,
                                          f32x16 (&acc)[C::FM][C::FN]) {
    constexpr int KK = C::BK / 16;
    constexpr int NF = C::FM + C::FN;           // fragments per K step
    constexpr int NRD = KK * NF;                // fragment reads per tile
    constexpr int NM = KK * C::FM * C::FN;      // MFMAs per tile
    constexpr int NG = C::LPW;                  // groups, one load each
    constexpr int MPG = NM / NG;                // MFMAs per group
    static_assert(NM % NG == 0 && NRD % MPG == 0 && NRD / MPG <= NG,
                  "group layout");
    __builtin_amdgcn_sched_barrier(0);
    if (q + 1 < ld.issued) wait_later<C>(ld.issued - q - 2);
    bulk_barrier();
    __builtin_amdgcn_sched_barrier(0);
    const BulkTile T = ld.prepare(smem);
    // (a stale stage is read when tile q + 1 does not exist; unused)
    const char *nst = smem + ((q + 1) % C::NS) * C::STAGE;
    const int r = lane & 31, half = lane >> 5;
    const int sw = swz_f<C>(r);
    const char *Aw = nst + wm * C::TM * C::RBY + r * C::RBY;
    const char *Bw = nst + C::BM * C::RBY + wn * C::TN * C::RBY + r * C::RBY;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        __builtin_amdgcn_sched_barrier(0);
        if (T.live) ld.load(T, g);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int x = g * MPG; x < (g + 1) * MPG; ++x) {
            if (x < NRD) {
                const int kk = x / NF, f = x % NF;
                const int co = ((2 * kk + half) ^ sw) << 4;
                if (f < C::FM)
                    nxt.a[kk][f] = *reinterpret_cast<const i32x4 *>(
                        Aw + f * 32 * C::RBY + co);
                else
                    nxt.b[kk][f - C::FM] = *reinterpret_cast<const i32x4 *>(
                        Bw + (f - C::FM) * 32 * C::RBY + co);
            }
        }
#pragma unroll
        for (int x = g * MPG; x < (g + 1) * MPG; ++x) {
            const int kk = x / (C::FM * C::FN), m = x % (C::FM * C::FN);
            const int i = m / C::FN, jj = m % C::FN;
            acc[i][jj] = mfma_bf16(cur.a[kk][i], cur.b[kk][jj], acc[i][jj]);
        }
#pragma unroll
        for (int x = g * MPG; x < (g + 1) * MPG; ++x) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if (x < NRD) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (T.live) ld.advance();
}

// Owned sub-tensors one after another; the K tiles of each are taken in
// pairs (register sets fixed at compile time), an odd last tile moves the
// next sub-tensor's first fragments back into set 0.
template <class C, class P>
__device__ __forceinline__ void run_bulk(const P &prov, char *smem) {
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform
    const int wm = wave / C::WN, wn = wave % C::WN;
    const int G = prov.n_prog(), total = prov.count();
    int t = program_slot(blockIdx.x, G);
    if (t >= total) return;
    BulkCursor<C, P> ld(prov, t, total, G, wave, lane);
    for (int s = 0; s < C::NS; ++s) ld.issue(smem);
    BulkFrags<C> F0, F1;
    wait_later<C>(ld.issued - 1);   // tile 0
    ring_barrier();
#pragma unroll
    for (int kk = 0; kk < C::BK / 16; ++kk)
        read_frags<C>(smem, wm, wn, lane, kk, F0.a[kk], F0.b[kk]);
    f32x16 acc[C::FM][C::FN];
    int q = 0;
    while (true) {
        const Job j = prov.job(t);
        const int nk = pp_tiles<C>(j.K);
        zero_acc<C>(acc);
        int kt = 0;
        for (; kt + 2 <= nk; kt += 2, q += 2) {
            bulk_iter<C, P>(ld, smem, q, wave, lane, wm, wn, F0, F1, acc);
            bulk_iter<C, P>(ld, smem, q + 1, wave, lane, wm, wn, F1, F0,
                            acc);
        }
        if (kt < nk) {
            bulk_iter<C, P>(ld, smem, q, wave, lane, wm, wn, F0, F1, acc);
            ++q;
            F0 = F1;
        }
        epilogue<C>(j, wm, wn, lane, acc, nullptr);
        t += G;
        if (t >= total) break;
    }
}

// ------------------------------------------------- register-staged ring
//
// Staged schedule (bf16, A and B both k-contiguous, 64-deep K tiles): the
// HBM reads of a K tile go into registers, two register sets deep, and
// reach LDS through ordinary 16-byte LDS stores into a ring of two stages.
// With four wavefronts of 128 x 128 outputs (accumulators in the AGPR
// half of the register file) the fragment reads per MFMA are a third
// lower than with eight wavefronts of 128 x 64, and every K tile is read
// from HBM two tile periods before the MFMAs need it: at the start of tile
// kt the registers of tile kt + 1 are stored into the free stage and the
// reads of tile kt + 3 are issued into them, while tile kt + 2 is still in
// flight in the other set.  One barrier per tile, before its last K step
// (as in the cross-tile schedule): by then every wavefront holds the
// tile's last fragments, and tile kt + 1 has been stored.
//
// Register-set indices must be compile-time constants, so tiles are taken
// in pairs.  Each owned sub-tensor starts its own pipeline (the reads of
// its first three tiles are issued after the previous sub-tensor's last
// MFMAs); K must be a whole number of K tiles.  Every tile issues its
// LDS stores and its reads unconditionally (reads past K are out of the
// buffer's range: zeros, no memory access), so that the compiler's
// load-counter bookkeeping sees the same order of outstanding reads on
// every path into the loop and waits only for the older register set.

// This wavefront's share of one K tile in registers: LPW chunks of 16
// bytes per lane, lane l of 1 KiB block rb holding the chunk that belongs
// at byte 16 l of the block (the layout of the direct loads).
template <class C>
struct StagedSet {
    i32x4 v[C::LPW];
};

// Where this wavefront's chunks of one K tile come from: a buffer
// resource per operand (rooted at the tile's first K column, formed in
// scalar registers without branches), one vector offset per operand (block
// i of the wavefront holds rows row + i * NW * RPK; the swizzle does not
// change over multiples of 16 rows, so every block of a lane reads the
// same logical chunk) and the scalar distance between blocks.
struct StagedSrc {
    __amdgpu_buffer_rsrc_t ra, rb;
    uint32_t va, vb;
    int sa, sb;
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t uniform_rsrc(
    const char *base, int64_t bytes) {
    const uint64_t p = reinterpret_cast<uint64_t>(base);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)p);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32));
    const uint32_t blo = __builtin_amdgcn_readfirstlane((uint32_t)bytes);
    const int32_t bhi = __builtin_amdgcn_readfirstlane((int32_t)(bytes >> 32));
    // clamp to [0, 2^31 - 1]: negative -> 0, at least 2^31 -> 2^31 - 1
    const uint32_t n = bhi < 0 ? 0u
                       : (bhi > 0 || blo > 0x7fffffffu) ? 0x7fffffffu : blo;
    return __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<void *>(((uint64_t)hi << 32) | lo), (short)0,
        (int)n, 0x00020000);
}

template <class C>
__device__ __forceinline__ StagedSrc staged_src(const Job &j, int k0,
                                                int wave, int lane) {
    static_assert((C::NW * C::RPK) % 16 == 0, "swizzle period");
    StagedSrc s;
    const int row = wave * C::RPK + lane / C::CPRW;
    const int kc = (lane % C::CPRW) ^ swz_f<C>(row);
    // tiles past K (the unconditional reads ahead of the last tiles) read
    // an empty buffer: zeros, no memory access
    const int64_t skip = (int64_t)k0 * C::ES;
    const bool live = k0 < j.K;
    s.ra = uniform_rsrc(j.a_row + skip, live ? j.a_rem - skip : 0);
    s.rb = uniform_rsrc(j.b_row + skip, live ? j.b_rem - skip : 0);
    s.va = (uint32_t)((row * j.lda + kc * C::EPC) * C::ES);
    s.vb = (uint32_t)((row * j.ldb + kc * C::EPC) * C::ES);
    s.sa = __builtin_amdgcn_readfirstlane(
        (int)(C::NW * C::RPK * j.lda * C::ES));
    s.sb = __builtin_amdgcn_readfirstlane(
        (int)(C::NW * C::RPK * j.ldb * C::ES));
    return s;
}

// Chunks [LO, HI) of this wavefront's share of a K tile into the register
// set (chunk c < NA is A block c, else B block c - NA).
template <class C, int LO, int HI>
__device__ __forceinline__ void staged_read(const StagedSrc &src,
                                            StagedSet<C> &s) {
    constexpr int NA = C::BM / C::RPK / C::NW;   // A blocks per wavefront
#pragma unroll
    for (int c = LO; c < HI; ++c) {
        if (c < NA)
            s.v[c] = __builtin_bit_cast(
                i32x4, __builtin_amdgcn_raw_buffer_load_b128(
                           src.ra, src.va, c * src.sa, 0));
        else
            s.v[c] = __builtin_bit_cast(
                i32x4, __builtin_amdgcn_raw_buffer_load_b128(
                           src.rb, src.vb, (c - NA) * src.sb, 0));
    }
}

template <class C, int LO, int HI>
__device__ __forceinline__ void staged_write(char *stage, int wave, int lane,
                                             const StagedSet<C> &s) {
    constexpr int NA = C::BM / C::RPK / C::NW;
#pragma unroll
    for (int c = LO; c < HI; ++c) {
        char *base = c < NA ? stage : stage + C::BM * C::RBY;
        const int i = c < NA ? c : c - NA;
        *reinterpret_cast<i32x4 *>(base + (i * C::NW + wave) * 1024 +
                                   lane * 16) = s.v[c];
    }
}

// MFMA slots of a K step that carry one of n evenly spaced instructions.
constexpr uint32_t spread_slots(int n, int slots, int shift) {
    uint32_t m = 0;
    for (int i = 0; i < n; ++i) m |= 1u << ((i * slots / n + shift) % slots);
    return m;
}

// The MFMAs of one K step with, slotted between them, the NREAD fragment
// reads (one after each of the first NREAD MFMAs) and the NWRITE LDS
// stores and NLOAD HBM reads issued just before in program order, spread
// evenly over the step so that the stores do not arrive at the LDS in a
// burst.
template <class C, int NREAD, int NWRITE, int NLOAD>
__device__ __forceinline__ void staged_mfma(const i32x4 (&af)[C::FM],
                                            const i32x4 (&bf)[C::FN],
                                            f32x16 (&acc)[C::FM][C::FN]) {
    constexpr int NM = C::FM * C::FN;
    constexpr uint32_t WS = spread_slots(NWRITE, NM, 0);
    constexpr uint32_t LS = spread_slots(NLOAD, NM, 1);
#pragma unroll
    for (int q = 0; q < NM; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (q < NREAD) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        if ((WS >> q) & 1u) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
        if ((LS >> q) & 1u) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    }
#pragma unroll
    for (int i = 0; i < C::FM; ++i)
#pragma unroll
        for (int jj = 0; jj < C::FN; ++jj)
            acc[i][jj] = mfma_bf16(af[i], bf[jj], acc[i][jj]);
}

// One K tile of the staged ring.  Tile kt (stage kt & 1) is contracted;
// set X holds tile kt + 1, which goes into the other stage over the first
// three K steps, each chunk's registers taking the matching chunk of tile
// kt + 3 right after; the other set holds tile kt + 2 (in flight).
template <class C>
__device__ __forceinline__ void staged_tile(
    const Job &j, char *smem, int kt, int nk, int wave, int lane, int wm,
    int wn, StagedSet<C> &X, i32x4 (&fa)[2][C::FM], i32x4 (&fb)[2][C::FN],
    f32x16 (&acc)[C::FM][C::FN]) {
    static_assert(C::BK / 16 == 4 && C::LPW == 16, "four K steps, 16 chunks");
    constexpr int NR = C::FM + C::FN;
    char *st = smem + (kt & 1) * C::STAGE;
    char *nx = smem + ((kt + 1) & 1) * C::STAGE;
    const StagedSrc src = staged_src<C>(j, (kt + 3) * C::BK, wave, lane);
    // one scheduling region per K step, so that each step's interleave
    // pattern takes that step's instructions
    read_frags<C>(st, wm, wn, lane, 1, fa[1], fb[1]);
    staged_write<C, 0, 6>(nx, wave, lane, X);
    staged_read<C, 0, 6>(src, X);
    staged_mfma<C, NR, 6, 6>(fa[0], fb[0], acc);
    __builtin_amdgcn_sched_barrier(0);
    read_frags<C>(st, wm, wn, lane, 2, fa[0], fb[0]);
    staged_write<C, 6, 11>(nx, wave, lane, X);
    staged_read<C, 6, 11>(src, X);
    staged_mfma<C, NR, 5, 5>(fa[1], fb[1], acc);
    __builtin_amdgcn_sched_barrier(0);
    read_frags<C>(st, wm, wn, lane, 3, fa[1], fb[1]);
    staged_write<C, 11, 16>(nx, wave, lane, X);
    staged_read<C, 11, 16>(src, X);
    staged_mfma<C, NR, 5, 5>(fa[0], fb[0], acc);
    // hand-over: tile kt + 1 is stored by every wavefront, nobody reads
    // tile kt any more (its last fragments are in registers)
    __builtin_amdgcn_sched_barrier(0);
    ring_barrier();
    __builtin_amdgcn_sched_barrier(0);
    if (kt + 1 < nk) read_frags<C>(nx, wm, wn, lane, 0, fa[0], fb[0]);
    staged_mfma<C, NR, 0, 0>(fa[1], fb[1], acc);
}

template <class C, class P>
__device__ __forceinline__ void run_staged(const P &prov, char *smem) {
    static_assert(C::BK / 16 % 2 == 0, "even number of K steps");
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform
    const int wm = wave / C::WN, wn = wave % C::WN;
    const int G = prov.n_prog(), total = prov.count();
    f32x16 acc[C::FM][C::FN];
    i32x4 fa[2][C::FM], fb[2][C::FN];
    StagedSet<C> S0, S1;
    for (int t = program_slot(blockIdx.x, G); t < total; t += G) {
        const Job j = prov.job(t);
        const int nk = (j.K + C::BK - 1) / C::BK;
        zero_acc<C>(acc);
        if (nk > 0) {
            // pipeline start: tiles 0 and 1 into the sets, tile 0 into
            // stage 0, tile 2 into set 0
            staged_read<C, 0, C::LPW>(staged_src<C>(j, 0, wave, lane), S0);
            staged_read<C, 0, C::LPW>(staged_src<C>(j, C::BK, wave, lane),
                                      S1);
            // the previous sub-tensor's reads of stage 0 ended at its
            // last hand-over barrier
            staged_write<C, 0, C::LPW>(smem, wave, lane, S0);
            staged_read<C, 0, C::LPW>(
                staged_src<C>(j, 2 * C::BK, wave, lane), S0);
            ring_barrier();
            read_frags<C>(smem, wm, wn, lane, 0, fa[0], fb[0]);
            int kt = 0;
            for (; kt + 1 < nk; kt += 2) {
                staged_tile<C>(j, smem, kt, nk, wave, lane, wm, wn, S1, fa,
                               fb, acc);
                staged_tile<C>(j, smem, kt + 1, nk, wave, lane, wm, wn, S0,
                               fa, fb, acc);
            }
            if (kt < nk)
                staged_tile<C>(j, smem, kt, nk, wave, lane, wm, wn, S1, fa,
                               fb, acc);
        }
        epilogue<C>(j, wm, wn, lane, acc, nullptr);
    }
}

template <class C>
__global__ __launch_bounds__(C::THREADS)
__attribute__((amdgpu_waves_per_eu(C::WPE, C::WPE))) void gemm_tiled_kernel(
    GemmArgs g) {
    extern __shared__ __align__(1024) char smem[];
    SingleProvider<C> p{g};
    if constexpr (C::PP)
        run_pingpong<C>(p, smem);
    else if constexpr (C::STG)
        run_staged<C>(p, smem);
    else if constexpr (C::BLK)
        run_bulk<C>(p, smem);
    else if constexpr (C::XT && C::NS == 5)
        run_direct_x5<C>(p, smem);
    else if constexpr (C::HALVES)
        run_direct_xh<C>(p, smem);
    else if constexpr (C::XT)
        run_direct_xt<C>(p, smem);
    else
        run_direct<C>(p, smem);
}

template <class C>
__global__ __launch_bounds__(C::THREADS)
__attribute__((amdgpu_waves_per_eu(C::WPE, C::WPE))) void gemm_grouped_kernel(
    const GroupProblem *__restrict__ tab, int n, int total, int G) {
    extern __shared__ __align__(1024) char smem[];
    GroupProvider<C> p{tab, n, total, G};
    if constexpr (C::PP)
        run_pingpong<C>(p, smem);
    else if constexpr (C::STG)
        run_staged<C>(p, smem);
    else if constexpr (C::BLK)
        run_bulk<C>(p, smem);
    else if constexpr (C::XT && C::NS == 5)
        run_direct_x5<C>(p, smem);
    else if constexpr (C::HALVES)
        run_direct_xh<C>(p, smem);
    else if constexpr (C::XT)
        run_direct_xt<C>(p, smem);
    else
        run_direct<C>(p, smem);
}

// Small outputs: one program per sub-tensor leaves compute units idle or
// with one wavefront each, and a K tile then takes about 0.45 us whatever the
// tile, the type or the depth of the ring: issue of the loads, LDS latency
// and a chain of dependent instructions, one after the other.  Here the W
// wavefronts of a program each contract whole K tiles (wave, wave + W, ...)
// of the whole sub-tensor, in a ring of their own that no other wavefront
// reads, so there is no barrier until the partial sub-tensors are summed, in
// the order of the wavefronts, through LDS.  C: the configuration of one
// wavefront.  bf16 64 x 4096 x 4096 9.4 us against 30, 1024^3 7.3 against
// 10.4, f32 512^3 5.7 against 14.7.
template <class C, int W, class P>
__device__ __forceinline__ void run_ksplit(const P &prov, char *smem) {
    static_assert(C::NW == 1 && C::NS == 2, "one wavefront, two stages");
    constexpr int NF = C::FM * C::FN;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    char *ring = smem + wave * C::NS * C::STAGE;
    const int G = prov.n_prog(), total = prov.count();
    for (int t = program_slot(blockIdx.x, G); t < total; t += G) {
        const Job j = prov.job(t);
        const int K = __builtin_amdgcn_readfirstlane(j.K);
        const int nk = (K + C::BK - 1) / C::BK;
        const int cnt = nk > wave ? (nk - wave + W - 1) / W : 0;
        const bool ragged = K % C::EPC != 0;
        auto k0 = [&](int i) { return (wave + i * W) * C::BK; };
        for (int i = 0; i < 2 && i < cnt; ++i)
            issue_direct<C>(j, ring + i * C::STAGE, k0(i), 0, lane);
        f32x16 acc[C::FM][C::FN];
        zero_acc<C>(acc);
        for (int i = 0; i < cnt; ++i) {
            char *stage = ring + (i & 1) * C::STAGE;
            if (i + 1 < cnt)
                wait_vmem_le<C::LPW>();
            else
                wait_vmem();
            asm volatile("" ::: "memory");
            if (ragged && wave + i * W == nk - 1) {
                fill_k_tail<C>(j, stage, k0(i), lane);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
            compute_stage<C>(stage, 0, 0, lane, acc, [](int, int) {});
            // the stage is free: its fragments have been read
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (i + 2 < cnt) issue_direct<C>(j, stage, k0(i + 2), 0, lane);
        }
        // partial sub-tensors over the rings, [fragment][register][lane]
        float *mine = reinterpret_cast<float *>(ring);
        constexpr int REGION = C::NS * C::STAGE / 4;
        static_assert(NF * 1024 <= REGION, "a partial sub-tensor per ring");
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                mine[(f * 16 + v) * 64 + lane] =
                    acc[f / C::FN][f % C::FN][v];
        __syncthreads();
        float *all = reinterpret_cast<float *>(smem);
        auto sum = [&](int e) {
            float x = all[e];
#pragma unroll
            for (int w = 1; w < W; ++w) x += all[w * REGION + e];
            return x;
        };
        f32x16 out[1][1];
        if constexpr (NF == W) {
            // a fragment per wavefront
            typedef Cfg<C::DTYPE, C::BM, C::BN, C::FM, C::FN, C::BNK,
                        C::CBF16, C::RBY, C::NS> E;
#pragma unroll
            for (int v = 0; v < 16; ++v)
                out[0][0][v] = sum((wave * 16 + v) * 64 + lane);
            epilogue<E>(j, wave / C::FN, wave % C::FN, lane, out, nullptr);
        } else {
            // 16 / W registers per wavefront, the first one stores
            static_assert(NF == 1 && 16 % W == 0, "one fragment");
#pragma unroll
            for (int v = 0; v < 16 / W; ++v) {
                const int e = (wave * (16 / W) + v) * 64 + lane;
                all[e] = sum(e);
            }
            __syncthreads();
            if (wave == 0) {
#pragma unroll
                for (int v = 0; v < 16; ++v) out[0][0][v] = all[v * 64 + lane];
                epilogue<C>(j, 0, 0, lane, out, nullptr);
            }
        }
        __syncthreads();
    }
}

template <class C, int W>
__global__ __launch_bounds__(W * 64)
__attribute__((amdgpu_waves_per_eu(W / 4, W / 4))) void gemm_ksplit_kernel(
    GemmArgs g) {
    extern __shared__ __align__(1024) char smem[];
    SingleProvider<C> p{g};
    run_ksplit<C, W>(p, smem);
}

template <class C, int W>
__global__ __launch_bounds__(W * 64)
__attribute__((amdgpu_waves_per_eu(W / 4, W / 4))) void
gemm_ksplit_grouped_kernel(const GroupProblem *__restrict__ tab, int n,
                           int total, int G) {
    extern __shared__ __align__(1024) char smem[];
    GroupProvider<C> p{tab, n, total, G};
    run_ksplit<C, W>(p, smem);
}

template <int DT, int T, int W, bool BNK, bool CBF16>
VariantEntry entry_ksplit() {
    typedef Cfg<DT, T, T, 1, 1, BNK, CBF16, 128, 2> C;
    VariantEntry e{};
    e.v.dtype = DT;
    e.v.bm = e.v.bn = T;
    e.v.bk = C::BK;
    e.v.stages = W * C::NS;       // of all its wavefronts
    e.v.sched = TG_SCHED_LOCKSTEP;
    e.v.wm = W; e.v.wn = 1;
    e.v.b_nk = BNK; e.v.c_bf16 = CBF16;
    e.kernel = reinterpret_cast<const void *>(&gemm_ksplit_kernel<C, W>);
    if constexpr (DT == TG_BF16)
        e.grouped =
            reinterpret_cast<const void *>(&gemm_ksplit_grouped_kernel<C, W>);
    e.threads = W * 64;
    e.smem = W * C::NS * C::STAGE;
    return e;
}

#define TG_KSPLIT(DT, T, W, BNK)                                              \
    entry_ksplit<DT, T, W, BNK, false>(), entry_ksplit<DT, T, W, BNK, true>()

template <class C>
VariantEntry make_entry() {
    VariantEntry e;
    e.v.dtype = C::DTYPE;
    e.v.bm = C::BM; e.v.bn = C::BN; e.v.bk = C::BK; e.v.stages = C::NS;
    e.v.sched = C::SCHED;
    e.v.wm = C::WM; e.v.wn = C::WN;
    e.v.b_nk = C::BNK; e.v.c_bf16 = C::CBF16;
    e.kernel = reinterpret_cast<const void *>(&gemm_tiled_kernel<C>);
    if constexpr (C::DTYPE == TG_BF16)
        e.grouped = reinterpret_cast<const void *>(&gemm_grouped_kernel<C>);
    e.threads = C::THREADS;
    e.smem = C::SMEM;
    return e;
}

#define TG_VARIANTS_FOR(DT, BM, BN, WM, WN, RBY, NS)                          \
    make_entry<Cfg<DT, BM, BN, WM, WN, false, false, RBY, NS>>(),             \
        make_entry<Cfg<DT, BM, BN, WM, WN, false, true, RBY, NS>>(),          \
        make_entry<Cfg<DT, BM, BN, WM, WN, true, false, RBY, NS>>(),          \
        make_entry<Cfg<DT, BM, BN, WM, WN, true, true, RBY, NS>>()

#define TG_VARIANTS_NK(DT, BM, BN, WM, WN, RBY, NS)                           \
    make_entry<Cfg<DT, BM, BN, WM, WN, true, false, RBY, NS>>(),              \
        make_entry<Cfg<DT, BM, BN, WM, WN, true, true, RBY, NS>>()

#define TG_VARIANTS_PP(DT, BM, BN, RBY, NS)                                   \
    make_entry<Cfg<DT, BM, BN, 2, 4, false, false, RBY, NS, TG_SCHED_PINGPONG>>(),         \
        make_entry<Cfg<DT, BM, BN, 2, 4, false, true, RBY, NS, TG_SCHED_PINGPONG>>(),      \
        make_entry<Cfg<DT, BM, BN, 2, 4, true, false, RBY, NS, TG_SCHED_PINGPONG>>(),      \
        make_entry<Cfg<DT, BM, BN, 2, 4, true, true, RBY, NS, TG_SCHED_PINGPONG>>()

#define TG_VARIANTS_XT_NK(DT, BM, BN, RBY, NS)                                \
    make_entry<Cfg<DT, BM, BN, 2, 4, true, false, RBY, NS, TG_SCHED_CROSS>>(), \
        make_entry<Cfg<DT, BM, BN, 2, 4, true, true, RBY, NS, TG_SCHED_CROSS>>()

#define TG_VARIANTS_XT_KN(DT, BM, BN, RBY, NS)                                \
    make_entry<Cfg<DT, BM, BN, 2, 4, false, false, RBY, NS, TG_SCHED_CROSS>>(), \
        make_entry<Cfg<DT, BM, BN, 2, 4, false, true, RBY, NS, TG_SCHED_CROSS>>()

#define TG_VARIANTS_BLK(DT, BM, BN, WM, WN, RBY, NS)                          \
    make_entry<Cfg<DT, BM, BN, WM, WN, true, false, RBY, NS, TG_SCHED_BULK>>(), \
        make_entry<Cfg<DT, BM, BN, WM, WN, true, true, RBY, NS, TG_SCHED_BULK>>()

#define TG_VARIANTS_STG(DT, BM, BN)                                           \
    make_entry<Cfg<DT, BM, BN, 2, 2, true, false, 128, 2, TG_SCHED_STAGED>>()

#define TG_VARIANTS_PP_NK(DT, BM, BN, RBY, NS)                                \
    make_entry<Cfg<DT, BM, BN, 2, 4, true, false, RBY, NS, TG_SCHED_PINGPONG>>(),          \
        make_entry<Cfg<DT, BM, BN, 2, 4, true, true, RBY, NS, TG_SCHED_PINGPONG>>()

// Table order is preference order: the first variant matching a request's
// dtype, partition, layout and output type is the default.
// The phased entries (gemm_phased.hip) come first.
std::vector<VariantEntry> all_entries() {
    int n;
    const VariantEntry *ph = phased_entries(&n);
    std::vector<VariantEntry> e(ph, ph + n);
    const VariantEntry entries[] = {
        TG_VARIANTS_FOR(TG_BF16, 256, 256, 2, 4, 128, 2),
        TG_VARIANTS_PP(TG_BF16, 256, 256, 64, 4),
        TG_VARIANTS_XT_NK(TG_BF16, 256, 256, 64, 4),
        TG_VARIANTS_XT_KN(TG_BF16, 256, 256, 64, 4),
        TG_VARIANTS_XT_NK(TG_BF16, 256, 256, 128, 3),
        TG_VARIANTS_XT_KN(TG_BF16, 256, 256, 128, 3),
        TG_VARIANTS_XT_NK(TG_BF16, 256, 256, 64, 5),
        TG_VARIANTS_XT_KN(TG_BF16, 256, 256, 64, 5),
        TG_VARIANTS_STG(TG_BF16, 256, 256),
        TG_VARIANTS_BLK(TG_BF16, 256, 256, 2, 2, 64, 4),
        TG_VARIANTS_BLK(TG_BF16, 256, 256, 2, 4, 64, 4),
        make_entry<Cfg<TG_BF16, 128, 128, 2, 4, false, false, 128, 4>>(),
        make_entry<Cfg<TG_BF16, 128, 128, 2, 4, false, true, 128, 4>>(),
        TG_VARIANTS_FOR(TG_BF16, 128, 128, 2, 2, 64, 4),
        TG_VARIANTS_FOR(TG_BF16, 128, 128, 2, 2, 128, 2),
        TG_VARIANTS_FOR(TG_BF16, 64, 64, 2, 2, 128, 2),
        TG_VARIANTS_FOR(TG_BF16, 64, 64, 2, 2, 128, 4),
        TG_VARIANTS_FOR(TG_BF16, 32, 32, 1, 1, 128, 2),
        TG_KSPLIT(TG_BF16, 32, 8, true), TG_KSPLIT(TG_BF16, 32, 8, false),
        TG_KSPLIT(TG_BF16, 64, 4, true), TG_KSPLIT(TG_BF16, 64, 4, false),
        // eight wavefronts: two per SIMD, one contracts while the other waits
        // (2048^3 141.5 us against 144.2 with four)
        TG_VARIANTS_FOR(TG_F32, 128, 128, 2, 4, 128, 2),
        TG_VARIANTS_FOR(TG_F32, 128, 128, 2, 2, 128, 2),
        TG_VARIANTS_FOR(TG_F32, 64, 64, 2, 2, 128, 2),
        TG_VARIANTS_FOR(TG_F32, 32, 32, 1, 1, 128, 2),
        TG_KSPLIT(TG_F32, 32, 8, true), TG_KSPLIT(TG_F32, 32, 8, false),
        TG_VARIANTS_NK(TG_FP8_E4M3, 256, 256, 2, 4, 128, 2),
        TG_VARIANTS_PP_NK(TG_FP8_E4M3, 256, 256, 64, 4),
        TG_VARIANTS_NK(TG_FP8_E4M3, 256, 256, 2, 4, 64, 4),
        TG_VARIANTS_NK(TG_FP8_E4M3, 128, 128, 2, 2, 128, 2),
        TG_VARIANTS_NK(TG_FP8_E4M3, 64, 64, 2, 2, 128, 2),
        TG_VARIANTS_NK(TG_FP8_E4M3, 64, 64, 2, 2, 128, 4),
        TG_VARIANTS_NK(TG_FP8_E4M3, 32, 32, 1, 1, 128, 2),
        TG_KSPLIT(TG_FP8_E4M3, 32, 8, true),
        TG_KSPLIT(TG_FP8_E4M3, 64, 4, true),
    };
    e.insert(e.end(), std::begin(entries), std::end(entries));
    return e;
}

const VariantEntry *table(int *count) {
    static const std::vector<VariantEntry> entries = all_entries();
    *count = (int)entries.size();
    return entries.data();
}

}  // namespace

int tiled_variant_count() {
    int n;
    table(&n);
    return n;
}

const TiledVariant &tiled_variant(int i) {
    int n;
    return table(&n)[i].v;
}

static hipError_t prepare_smem(const VariantEntry &e) {
    static LdsRequest request[128];
    int n;
    const int idx = (int)(&e - table(&n));
    LdsRequest once;
    return (idx < 128 ? request[idx] : once)({e.kernel, e.grouped, e.planes},
                                             e.smem);
}

const void *tiled_kernel(int variant) {
    int n;
    return table(&n)[variant].kernel;
}

bool tiled_planes(int variant) {
    int n;
    return table(&n)[variant].planes != nullptr;
}

hipError_t launch_tiled(int variant, const GemmArgs &args, hipStream_t st) {
    int n;
    const VariantEntry &e = table(&n)[variant];
    hipError_t err = prepare_smem(e);
    if (err != hipSuccess) return err;
    void *params[] = {const_cast<GemmArgs *>(&args)};
    return hipLaunchKernel(args.kp ? e.planes : e.kernel,
                           dim3(args.s.n_prog), dim3(e.threads), params,
                           e.smem, st);
}

hipError_t launch_grouped(int variant, int n_problems, int total_tiles,
                          int n_prog, const void *table_dev, hipStream_t st) {
    int n;
    const VariantEntry &e = table(&n)[variant];
    if (!e.grouped) return hipErrorInvalidValue;
    hipError_t err = prepare_smem(e);
    if (err != hipSuccess) return err;
    const GroupProblem *tab = static_cast<const GroupProblem *>(table_dev);
    int np = n_problems, total = total_tiles, G = n_prog;
    void *params[] = {&tab, &np, &total, &G};
    return hipLaunchKernel(e.grouped, dim3(G), dim3(e.threads), params,
                           e.smem, st);
}

// (asked of the runtime once per variant: it depends on the compiled kernel
// and the architecture alone)
int tiled_occupancy(int variant) {
    static std::atomic<int> known[128];
    int n;
    const VariantEntry &e = table(&n)[variant];
    const bool keep = variant >= 0 && variant < 128;
    if (keep)
        if (const int k = known[variant].load(std::memory_order_relaxed))
            return k;
    int blocks = 0;
    if (prepare_smem(e) != hipSuccess) return 1;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &blocks, e.kernel, e.threads, e.smem) != hipSuccess ||
        blocks < 1)
        return 1;
    if (keep) known[variant].store(blocks, std::memory_order_relaxed);
    return blocks;
}

}  // namespace tg
