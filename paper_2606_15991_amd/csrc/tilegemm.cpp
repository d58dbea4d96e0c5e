// tilegemm.cpp -- host side of the C ABI: argument validation, the
// ownership checks of tile_partition_check, configuration choice, the
// program map, and kernel dispatch.  No call here allocates device memory.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <unordered_map>
#include <vector>

#include "host_internal.hpp"
#include "tg_internal.hpp"
#include "tg_elementwise.hpp"

using namespace tg;

namespace {

thread_local std::string g_err;

tg_status fail(tg_status st, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return st;
}

tg_status hip_fail(hipError_t e, const char *what) {
    return fail(TG_E_HIP, "%s: %s", what, hipGetErrorString(e));
}

int esize(int dt) {
    switch (dt) {
    case TG_F32: return 4;
    case TG_BF16: return 2;
    case TG_FP8_E4M3: return 1;
    default: return 0;
    }
}

struct Range {
    uintptr_t lo, hi;  // [lo, hi); empty when lo == hi
};

Range byte_range(const void *data, int64_t rows, int64_t cols, int64_t ld,
                 int es) {
    Range r{(uintptr_t)data, (uintptr_t)data};
    if (rows > 0 && cols > 0)
        r.hi = r.lo + (uintptr_t)(((rows - 1) * ld + cols) * es);
    return r;
}

bool intersect(const Range &a, const Range &b) {
    if (a.lo == a.hi || b.lo == b.hi) return false;
    return a.lo < b.hi && b.lo < a.hi;
}

tg_status check_in(const tg_in *d, const char *name) {
    if (!d) return fail(TG_E_ARG, "%s: NULL descriptor", name);
    if (esize(d->dtype) == 0)
        return fail(TG_E_ARG, "%s: unknown dtype %d", name, d->dtype);
    if (d->rows < 0 || d->cols < 0)
        return fail(TG_E_ARG, "%s: negative size", name);
    if (d->trans != 0 && d->trans != 1)
        return fail(TG_E_ARG, "%s: trans must be 0 or 1", name);
    if (d->rows > 0 && d->cols > 0 && !d->data)
        return fail(TG_E_ARG, "%s: NULL data", name);
    if (d->rows > 1 && d->ld < d->cols)
        return fail(TG_E_SHAPE, "%s: ld %lld < cols %lld", name,
                    (long long)d->ld, (long long)d->cols);
    if (d->ld < 0) return fail(TG_E_SHAPE, "%s: negative ld", name);
    return TG_OK;
}

tg_status check_out(const tg_out *d, bool need_partition) {
    if (!d) return fail(TG_E_ARG, "C: NULL descriptor");
    if (d->dtype != TG_F32 && d->dtype != TG_BF16)
        return fail(TG_E_ARG, "C: dtype must be TG_F32 or TG_BF16");
    if (d->rows < 0 || d->cols < 0) return fail(TG_E_ARG, "C: negative size");
    if (d->rows > 0 && d->cols > 0 && !d->data)
        return fail(TG_E_ARG, "C: NULL data");
    if (need_partition && (d->bm <= 0 || d->bn <= 0))
        return fail(TG_E_ARG, "C: partition %d x %d must be positive", d->bm,
                    d->bn);
    if (d->bm < 0 || d->bn < 0) return fail(TG_E_ARG, "C: negative partition");
    if (d->rows > 1 && d->ld < d->cols)
        return fail(TG_E_SHAPE, "C: ld %lld < cols %lld", (long long)d->ld,
                    (long long)d->cols);
    if (d->ld < 0) return fail(TG_E_SHAPE, "C: negative ld");
    return TG_OK;
}

// Program-map rules: every id on the grid, no sub-tensor twice, none missed.
tg_status check_map(int64_t tiles, int32_t n_prog, const int32_t *offs,
                    const int32_t *ids) {
    if (n_prog < 0) return fail(TG_E_ARG, "negative program count");
    if (n_prog == 0) return TG_OK;
    if (!offs || !ids) return fail(TG_E_ARG, "NULL program map");
    if (offs[0] != 0) return fail(TG_E_ARG, "program map must start at 0");
    // reused per thread: after the first call of a size, checking
    // allocates nothing
    static thread_local std::vector<uint8_t> seen;
    seen.assign((size_t)tiles, 0);
    for (int32_t p = 0; p < n_prog; ++p) {
        if (offs[p + 1] < offs[p])
            return fail(TG_E_ARG, "program %d: decreasing offsets", p);
        for (int32_t q = offs[p]; q < offs[p + 1]; ++q) {
            int64_t t = ids[q];
            if (t < 0 || t >= tiles)
                return fail(TG_E_ARG, "program %d: sub-tensor %lld off the grid",
                            p, (long long)t);
            if (seen[(size_t)t])
                return fail(TG_E_OVERLAP,
                            "sub-tensor %lld owned by two programs (second: %d)",
                            (long long)t, p);
            seen[(size_t)t] = 1;
        }
    }
    for (int64_t t = 0; t < tiles; ++t)
        if (!seen[(size_t)t])
            return fail(TG_E_NOCOVER, "sub-tensor %lld owned by no program",
                        (long long)t);
    return TG_OK;
}

tg_status check_alias(const tg_in *ins, int32_t n_in, const tg_out *out) {
    Range ro = byte_range(out->data, out->rows, out->cols, out->ld,
                          esize(out->dtype));
    for (int32_t i = 0; i < n_in; ++i) {
        Range ri = byte_range(ins[i].data, ins[i].rows, ins[i].cols, ins[i].ld,
                              esize(ins[i].dtype));
        if (intersect(ro, ri))
            return fail(TG_E_ALIAS, "output shares bytes with input %d", i);
    }
    return TG_OK;
}

// ------------------------------------------------------------- device info

int device_cus() {
    static std::mutex mu;
    static std::unordered_map<int, int> cache;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    std::lock_guard<std::mutex> lk(mu);
    auto it = cache.find(dev);
    if (it != cache.end()) return it->second;
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount,
                              dev) != hipSuccess)
        cus = 0;
    cache[dev] = cus;
    return cus;
}

// --------------------------------------------------------------- problem

struct Problem {
    int64_t M, N, K;
    int a_dt, b_dt;
    bool b_nk;
    bool c_bf16;
    int precision;
    bool scaled;       // row or column scales given
};

tg_status describe(const tg_in *A, const tg_in *B, const tg_out *C,
                   const tg_opts *o, Problem &p) {
    tg_status st;
    if ((st = check_in(A, "A")) != TG_OK) return st;
    if ((st = check_in(B, "B")) != TG_OK) return st;
    if ((st = check_out(C, false)) != TG_OK) return st;
    if (A->trans) return fail(TG_E_UNSUPPORTED, "A must not be transposed");
    p.M = A->rows;
    p.K = A->cols;
    p.b_nk = B->trans == 1;
    int64_t bk = p.b_nk ? B->cols : B->rows;
    p.N = p.b_nk ? B->rows : B->cols;
    if (bk != p.K)
        return fail(TG_E_SHAPE, "A is %lld x %lld but B has K = %lld",
                    (long long)A->rows, (long long)A->cols, (long long)bk);
    if (C->rows != p.M || C->cols != p.N)
        return fail(TG_E_SHAPE, "C is %lld x %lld, expected %lld x %lld",
                    (long long)C->rows, (long long)C->cols, (long long)p.M,
                    (long long)p.N);
    if (p.M > INT32_MAX || p.N > INT32_MAX || p.K > INT32_MAX)
        return fail(TG_E_SHAPE, "dimension exceeds 2^31 - 1");
    p.a_dt = A->dtype;
    p.b_dt = B->dtype;
    p.c_bf16 = C->dtype == TG_BF16;
    p.precision = o ? o->precision : TG_PREC_NATIVE;
    p.scaled = o && (o->scale_a || o->scale_b);
    if (p.precision < TG_PREC_NATIVE || p.precision > TG_PREC_BF16X6)
        return fail(TG_E_ARG, "unknown precision %d", p.precision);
    bool same = p.a_dt == p.b_dt;
    bool w8 = p.a_dt == TG_BF16 && p.b_dt == TG_FP8_E4M3;
    if (!same && !w8)
        return fail(TG_E_DTYPE, "dtype pair (%d, %d) not provided", p.a_dt,
                    p.b_dt);
    if (p.precision != TG_PREC_NATIVE &&
        (p.a_dt != TG_F32 || p.b_dt != TG_F32))
        return fail(TG_E_DTYPE, "split precision needs f32 A and B");
    return TG_OK;
}

// A single row has no stride, and check_in takes any for it; the kernels size
// their buffers by it.
tg_in row_stride(const tg_in &d) {
    tg_in r = d;
    if (r.rows <= 1 && r.ld < r.cols) r.ld = r.cols;
    return r;
}

bool aligned16(const void *p) { return ((uintptr_t)p & 15u) == 0; }

// Can the tiled kernel take this operand layout?
bool tiled_ok(const Problem &p, const tg_in *A, const tg_in *B,
              const tg_out *C, int dt) {
    int es = esize(dt);
    int epc = 16 / es;
    if (p.a_dt != p.b_dt) return false;
    if (dt == TG_FP8_E4M3 && !p.b_nk) return false;
    if (!aligned16(A->data) || !aligned16(B->data)) return false;
    // row starts must stay 16-byte aligned (a single row has no stride)
    if ((A->rows > 1 && (A->ld * es) % 16) || (B->rows > 1 && (B->ld * es) % 16))
        return false;
    // bf16 / e4m3 take any K (the straddling chunk is filled element-wise);
    // f32 needs whole 16-byte chunks
    if (dt == TG_F32 && p.K % epc) return false;
    if (!p.b_nk && (p.N % epc)) return false;
    // the kernels address a sub-tensor with 32-bit byte offsets: 256 rows of
    // any operand (and of C in binary32) must span less than 2^31 bytes
    const int64_t lim = (int64_t)1 << 31;
    if (row_stride(*A).ld * es * 256 >= lim ||
        row_stride(*B).ld * es * 256 >= lim)
        return false;
    if (C->ld * 4 * 256 >= lim) return false;
    return true;
}

bool skinny_ok(const Problem &p, const tg_in *A, const tg_in *B) {
    if (p.M > 16 || !p.b_nk || p.a_dt != TG_BF16) return false;
    if (p.b_dt != TG_BF16 && p.b_dt != TG_FP8_E4M3) return false;
    if (!aligned16(A->data) || !aligned16(B->data)) return false;
    if ((A->rows > 1 && (A->ld * 2) % 16) ||
        (B->rows > 1 && (B->ld * esize(p.b_dt)) % 16))
        return false;
    return true;
}

// First tiled variant matching the request; zero fields match anything.
// Ping-pong variants have no tail fill for a 16-byte chunk straddling K:
// pp_ok is false when K is not a multiple of the chunk.  Bulk-read
// variants need K a whole number of their 32-deep K tiles (k32_ok).  Staged variants
// need K a whole number of their K tiles (k_tiles_ok: K % 64 == 0 for
// bf16) and apply no scales.
int find_variant(int dt, int bm, int bn, int wm, int wn, int bk, int stages,
                 int sched, bool b_nk, bool c_bf16, bool pp_ok,
                 bool scaled = false, bool k_tiles_ok = false,
                 bool k32_ok = false) {
    int n = tiled_variant_count();
    for (int i = 0; i < n; ++i) {
        const TiledVariant &v = tiled_variant(i);
        if (v.sched == TG_SCHED_PINGPONG && !pp_ok) continue;
        if (v.sched == TG_SCHED_BULK && !k32_ok) continue;
        if (v.sched == TG_SCHED_STAGED && (scaled || !k_tiles_ok)) continue;
        if (v.dtype == dt && v.bm == bm && v.bn == bn && v.b_nk == b_nk &&
            v.c_bf16 == c_bf16 && (wm == 0 || v.wm == wm) &&
            (wn == 0 || v.wn == wn) && (bk == 0 || v.bk == bk) &&
            (stages == 0 || v.stages == stages) &&
            (sched == 0 || v.sched == sched))
            return i;
    }
    return -1;
}

bool chunk_multiple(int64_t K, int dt) { return (K * esize(dt)) % 16 == 0; }

int64_t tiles_of(int64_t M, int64_t N, int s) {
    return ((M + s - 1) / s) * ((N + s - 1) / s);
}

// Sub-tensor of a configuration that names wavefronts, stages, bk or a
// schedule but no size: the largest square one that still gives every compute
// unit close to one.  (Which of those exist depends on the size, so this rule
// does not move with the defaults below: what it accepts stays accepted.)
int named_tile(int dt, int64_t M, int64_t N, int cus) {
    if (cus <= 0) cus = 256;
    for (int s : {256, 128, 64})
        if ((dt != TG_F32 || s < 256) &&
            tiles_of(M, N, s) * 4 >= (int64_t)cus * 3)
            return s;
    return 32;
}

// Default sub-tensor of a tiled product, and LDS stages where they matter
// (0: the variant table's first).  With t(s) sub-tensors of s x s on `cus`
// compute units, measured in a graph of one launch each (B stored N x K):
//  256 (phased) where 128 takes more than two programs per compute unit, as
//      many as are resident: bf16 3072^3 (t(128) = 576) 61 us against 97, 2048
//      x 5120 x 5120 (640) 96 against 154; but 4096 x 2048 x 2048 (512) 46
//      against 42, e4m3 27.6 against 24.2, 2816 x 2560 x 3000 (440) 63 against
//      59, 2048^3 42 against 27.  Not for outputs of at most 128 rows or
//      columns (64 x 65536 x 512: 19 against 15 with 64);
//  128: one round in the phased kernel (B stored N x K): bf16 from a quarter
//      of the compute units on, 256 x 8192 x 4096 (t(128) = 128) 30.5 us
//      against 39.4 with 64, 512 x 5120 x 5120 (160) 37.6 against 64.8, 1280^3
//      (100) 13.2 against 15.0 (but with few K tiles behind: 8982 x 112 (71) x
//      64 4.7 against 4.1, level at x 384);
//      e4m3, whose 64 reads half the bytes, from eleven in twenty on: 512 x
//      5120 x 5120 24.4 against 28.9, 1536^3 (144) 10.2 against 10.7, but
//      1024 x 1536 x 4096 (96) 20.3 against 18.5.  bf16 K x N (eight
//      wavefronts in step, four stages) from eleven in twenty: 1536^3 18.7
//      against 22.4, 256 x 8192 x 4096 41.0 against 38.8.  Past one round two
//      programs of two stages per compute unit (rounds_128);
//  64: four stages where all programs are then resident at once (two per
//      compute unit) and there are at least 36 K tiles: bf16 K x N 256 x 8192
//      x 4096 38.8 us against 44.6; but 1536^3 (t(64) = 576) 31.5 against
//      22.6 and e4m3 1280^3 (10 K tiles) 8.6 against 8.2;
//  32 where 64 leaves a quarter of the compute units idle.
// f32 is bound by the matrix instructions alone, so the busiest compute unit
// decides: ceil(t / cus) rounds at 36 us (64) and 128 us (128) for K = 2048:
//  128 where two of its rounds take no longer than seven of 64: 2048^3 (1 and
//      4 rounds) 141 us against 145, 4096^3 (4 and 16) 1025 against 1098;
//  64  else: 3072^3 (9 rounds, 128: 3) 475 us against 578, 512 x 5120 x 5120
//      (3, 1) 275 against 342, 1000 x 3000 x 2000 (3, 1) 112 against 138;
//  32 is never ahead (512^3 16.5 us against 15.6, 130 x 3000 x 256 10.0
//      against 9.7) and is left to outputs of at most 32 rows or columns.
// First of all, outputs of at most one sub-tensor per compute unit take the
// programs whose wavefronts share K (wm = 8 of 32 x 32, 4 of 64 x 64), from
// four and eight K tiles on:
//  32  t(32) <= cus: bf16 300 x 300 x 8192 14.4 us against 57 (64, four
//      stages), 64 x 4096 x 4096 9.4 against 30; e4m3 512^3 (four K tiles)
//      3.6 against 4.1, but 128^3 (one) 3.2 against 2.9; f32 up to three
//      rounds, from four, eight and sixteen K tiles on: 512^2 x 128 (t(32) =
//      256) 0.73 of the time of the best other, 640^2 (400) x 192 1.04, x 256
//      0.89, 800^2 (625) x 384 1.05, x 512 0.97, x 2048 37 us against 50, but
//      1024^3 (1024) 28.8 against 26.9; 32 rows or columns always from four
//      on (24576 x 32 x 128 in three rounds 1.4 times 32, which is 1.5 times
//      what binary32 took in its first form);
//  64  t(64) <= cus: bf16 1024^3 7.3 us against 10.4, 1024^2 x 4096 15.8
//      against 30.6 (128), 256 x 2560 x 2560 10.7 against 20.4; e4m3 1024^3
//      (eight) 5.8 against 6.1, 768^3 (six) 5.2 against 5.1.
struct DefaultTile {
    int size, stages, wm = 0;
};
DefaultTile default_tile(int dt, int64_t M, int64_t N, int64_t K, bool b_nk,
                         int cus) {
    if (cus <= 0) cus = 256;
    const auto t = [&](int s) { return tiles_of(M, N, s); };
    if (dt == TG_F32) {
        const auto rounds = [&](int s) { return (t(s) + cus - 1) / cus; };
        const int64_t side = std::min(M, N), r32 = rounds(32);
        if (r32 <= 3 && K >= (side <= 32 ? 128 : 64 << r32))
            return {32, 16, 8};
        if (side <= 32) return {32, 0};
        return {2 * rounds(64) >= 7 * rounds(128) ? 128 : 64, 0};
    }
    const int64_t nk = K * esize(dt) / 128, side = std::min(M, N);
    if (t(32) <= cus && nk >= 4) return {32, 16, 8};
    if (t(64) <= cus && nk >= 8) return {64, 8, 4};
    if (side > 128 && t(128) > 2 * cus) return {256, 0};
    if (side > 64 &&
        t(128) * 20 >= (int64_t)cus * (dt == TG_BF16 && b_nk ? 5 : 11))
        return {128, 0};      // (stages: rounds_128)
    const bool deep = t(64) <= 2 * cus && nk >= 36;
    if (deep || t(64) * 4 >= (int64_t)cus * 3) return {64, deep ? 4 : 2};
    return {32, 0};
}

struct Launch {
    tg_config cfg;
    int variant;       // tiled kernel index, or -1
    int gemm_dt;       // dtype the contraction reads (bf16 for split modes)
    int64_t Kc;        // contraction length seen by the kernel
    int32_t sps;       // decode kernel: K steps per split
    int32_t gm, gn;    // simple kernel: sub-tensors per program
    bool mixed;        // simple kernel: bf16 x e4m3 on the phased kernel
    int32_t stream;    // decode kernel: skinny_stream's answer
    Sched s;
};

size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

// Workspace of a decode product split over `splitk` programs per
// sub-tensor: partial tiles [splitk][M][N] binary32, then (fused
// normalisation) partial sums of squares [splitk][M].
size_t skinny_ws_bytes(int64_t splitk, int64_t M, int64_t N, bool norm) {
    if (splitk <= 1) return 0;
    return up256((size_t)splitk * M * N * 4) +
           (norm ? up256((size_t)splitk * M * 4) : 0);
}

// Decode kernel geometry: K steps (32 bf16 or 64 e4m3 weights per lane
// group) and super-steps (eight 16-byte weight loads per lane).
struct SkinnyGeo {
    int64_t kstep, unroll, nsteps, supers;
};
SkinnyGeo skinny_geo(const Problem &p, int bn) {
    SkinnyGeo g;
    g.kstep = p.b_dt == TG_BF16 ? 32 : 64;
    g.unroll = bn > 16 ? 4 : 8;   // two row tiles: four K steps of two
    g.nsteps = (p.K + g.kstep - 1) / g.kstep;
    g.supers = (g.nsteps + g.unroll - 1) / g.unroll;
    return g;
}

// Decode columns per program that deal N evenly over whole rounds of the
// compute units: N / (ncu r) for the fewest rounds r that bring it to at
// most 32 columns and divide N exactly (else ceil(N / (ncu r)) for the
// fewest rounds); 0 where that leaves fewer than 8 columns per program.
int32_t balanced_bn(int64_t N, int64_t ncu) {
    const int64_t r0 = (N + 32 * ncu - 1) / (32 * ncu);
    for (int64_t r = r0; r < r0 + 4; ++r)
        if (N % (ncu * r) == 0 && N / (ncu * r) >= 8)
            return (int32_t)(N / (ncu * r));
    const int64_t bn = (N + ncu * r0 - 1) / (ncu * r0);
    return bn >= 8 && bn <= 32 ? (int32_t)bn : 0;
}

// Splits that get K work when `splitk` are asked for: each split takes
// ceil(supers / splitk) whole super-steps.
int32_t effective_splitk(int64_t supers, int64_t splitk, int64_t *per) {
    if (supers <= 0 || splitk <= 1) {
        if (per) *per = supers > 0 ? supers : 1;
        return 1;
    }
    const int64_t q = (supers + splitk - 1) / splitk;
    if (per) *per = q;
    return (int32_t)((supers + q - 1) / q);
}

int32_t simple_blocks_m(const Launch &L) {
    return (L.s.tiles_m + L.gm - 1) / L.gm;
}

// Sub-tensors per program of the simple kernel: 2 x 2 of the default 64 x 64
// ones (a 128 x 128 block of eight wavefronts, half the operand traffic per
// product) where that leaves a program for at least every second compute
// unit.  Measured, 2 x 2 against 1 x 1: e4m3 weights 512 x 5120 x 5112 (160 such
// programs) 55 us against 64, stored K x N 47 against 57, bf16 2000 x 2003 x
// 1003 (256) 27 against 40, 512 x 5120 x 5001 (160) 88 against 103.  Near the
// line, at 132 programs, bf16 1400 x 1500 x 1003 is behind, 27.8 against 25.0,
// binary32 x 1001 73 against 58; the mixed form needs the blocks there.  Below
// it 1111 x 1531 x 1003 (108) ran 26 us in blocks, 21.7 in 432 programs.
void simple_group(Launch &L, const tg_config &cfg, int cus) {
    L.gm = L.gn = 1;
    if (cfg.bm != 64 || cfg.bn != 64) return;
    if (cus <= 0) cus = 256;
    const int64_t progs = (int64_t)((L.s.tiles_m + 1) / 2) *
                          ((L.s.tiles_n + 1) / 2);
    if (2 * progs >= cus) L.gm = L.gn = 2;
}

// bf16 rows by e4m3 weights in blocks of 2 x 2 sub-tensors: the phased kernel
// takes what its 16-byte direct loads can (512 x 5120 x 5120 44 us against
// 49 through registers).
bool mixed_ok(const Problem &p, const tg_in *A, const tg_in *B,
              const tg_out *C, const Launch &L) {
    const int64_t lim = (int64_t)1 << 31;
    const int64_t lda = row_stride(*A).ld, ldb = row_stride(*B).ld;
    return p.a_dt == TG_BF16 && p.b_dt == TG_FP8_E4M3 && p.b_nk &&
           L.gm == 2 && L.gn == 2 && L.cfg.bm == 64 && L.cfg.bn == 64 &&
           p.K > 0 && p.K % 16 == 0 && aligned16(A->data) &&
           aligned16(B->data) && (A->rows == 1 || lda % 8 == 0) &&
           (B->rows == 1 || ldb % 16 == 0) && lda * 2 * 256 < lim &&
           ldb * 256 < lim && C->ld * 4 * 256 < lim;
}

// `have`: workspace bytes the caller supplies; the default K split of a
// decode product is reduced until its workspace fits.
tg_status choose_explicit(const Problem &p, const tg_in *A, const tg_in *B,
                          const tg_out *C, const tg_config *uc, Launch &L,
                          size_t have, bool norm = false) {
    tg_config cfg{};
    if (uc) cfg = *uc;
    if (cfg.kind < TG_KIND_AUTO || cfg.kind > TG_KIND_SIMPLE)
        return fail(TG_E_ARG, "unknown kernel kind %d", cfg.kind);
    int np = p.precision == TG_PREC_BF16X3 ? 3
             : p.precision == TG_PREC_BF16X6 ? 6 : 1;
    L.gemm_dt = np > 1 ? TG_BF16 : p.a_dt;
    L.Kc = p.K * np;
    // the partition of C, when given, fixes the sub-tensor shape
    if (C->bm > 0 || C->bn > 0) {
        if (C->bm <= 0 || C->bn <= 0)
            return fail(TG_E_ARG, "C partition %d x %d: both must be set",
                        C->bm, C->bn);
        if (cfg.bm && cfg.bm != C->bm)
            return fail(TG_E_ARG, "config bm %d != partition bm %d", cfg.bm,
                        C->bm);
        if (cfg.bn && cfg.bn != C->bn)
            return fail(TG_E_ARG, "config bn %d != partition bn %d", cfg.bn,
                        C->bn);
        cfg.bm = C->bm;
        cfg.bn = C->bn;
    }
    // split precisions run the tiled bf16 kernel on the plane operands,
    // whose layout the library lays out itself (always aligned)
    bool t_ok = np > 1 ? ((p.K * np) % 8 == 0 && (p.b_nk || p.N % 8 == 0) &&
                          p.K * np * 2 * 256 < ((int64_t)1 << 31) &&
                          C->ld * 4 * 256 < ((int64_t)1 << 31))
                       : tiled_ok(p, A, B, C, p.a_dt);
    bool s_ok = np == 1 && skinny_ok(p, A, B);
    if (cfg.kind == TG_KIND_AUTO) {
        if (s_ok && (cfg.bm == 0 || (cfg.bm >= p.M && cfg.bm <= 16)) &&
            cfg.bn >= 0 && cfg.bn <= 32)
            cfg.kind = TG_KIND_SKINNY;
        else if (t_ok && (cfg.bm == 0 ||
                          find_variant(L.gemm_dt, cfg.bm, cfg.bn, cfg.wm,
                                       cfg.wn, cfg.bk, cfg.stages, cfg.sched,
                                       p.b_nk, p.c_bf16,
                                       chunk_multiple(L.Kc, L.gemm_dt),
                                       p.scaled, L.Kc % 64 == 0,
                                       L.Kc % 32 == 0) >= 0))
            cfg.kind = TG_KIND_TILED;
        else
            cfg.kind = TG_KIND_SIMPLE;
    }
    int cus = device_cus();
    L.variant = -1;
    L.mixed = false;
    L.stream = 0;
    if (cfg.kind == TG_KIND_SKINNY) {
        if (!s_ok)
            return fail(TG_E_UNSUPPORTED,
                        "decode kernel needs M <= 16, bf16 A, bf16/e4m3 B "
                        "stored N x K, aligned 16-byte rows");
        if (cfg.bm == 0) cfg.bm = 16;
        // the decode defaults assume MI355X's 256 compute units where the
        // device cannot be asked (host-only planning)
        const int64_t ncu = cus > 0 ? cus : 256;
        // (The rules below were measured on the plain form of the kernel.
        // Where the streaming form runs instead, their programs' columns are
        // dealt to one workgroup per compute unit and ksplit is not used;
        // the even widths suit it too.)
        // One round of programs, one per compute unit: where N / ncu is 8 to
        // 32 columns, programs of that many columns fill the machine with
        // no K split and so no merge launch.  Measured on (M, N, K) =
        // (1 and 8, 5120, 5120) and (1, 5120, 25600), bf16 and e4m3 cold
        // weights: 3.5-17 % faster than 16-column programs with the best
        // K split (for (1, 51200, 5120), eight rounds of 25 columns lose
        // to 16-column programs, so only the one-round case takes it).
        const int32_t bal = balanced_bn(p.N, ncu);
        const bool one_round = cfg.bn == 0 && cfg.splitk <= 1 && bal > 0 &&
                               p.N <= 32 * ncu;
        // Several rounds with more than four activation rows: programs of
        // the even width and one wavefront each, so that all of them are
        // resident at once (eight per compute unit at N = 51200) with no
        // K split.  Measured at (8 and 16, 51200, 5120): 4-17 % faster
        // than 16- or 32-column programs of four wavefronts, bf16 and
        // e4m3; at (8, 16384 and 32768, 4096) within -14..+4 %.
        const bool resident = cfg.bn == 0 && cfg.splitk <= 1 && bal > 0 &&
                              !one_round && p.M > 4;
        if (one_round || resident) cfg.bn = bal;
        // bf16 weights, up to four activation rows, K up to 8192: where the
        // one-round width needs two row tiles (more than 16 columns), half
        // of it in one row tile, two programs per compute unit of two
        // wavefronts each (both resident).  Measured at N = 5120, 6144 and
        // 8192 (K 4096-8192): 4-18 % faster; at (1, 5120, 25600) 9 %
        // slower, and where the one-round width is 16 or less (N = 4096)
        // 7 % slower, hence the bounds.  Not for the fused normalisation,
        // whose programs each stage the normalisation weights of their K
        // range: twice the programs cost more than they gain (decode
        // layer 21.0 against 19.9 us).
        const bool halves = one_round && !norm && p.b_dt == TG_BF16 &&
                            p.M <= 4 && p.K <= 8192 && bal > 16;
        if (halves) cfg.bn = (bal + 1) / 2;
        if (cfg.bn == 0) {
            // 32-column programs (each activation chunk serves two weight
            // rows) for e4m3 weights with more than four activation rows,
            // or three or four over long sweeps; measured on the decode
            // shapes with cold weights
            const bool wide =
                p.b_dt == TG_FP8_E4M3 &&
                (p.M > 4 || (p.M > 2 && (p.N + 15) / 16 >= 4 * ncu));
            cfg.bn = wide ? 32 : 16;
        }
        if (cfg.bm < p.M || cfg.bm > 16 || cfg.bn < 1 || cfg.bn > 32)
            return fail(TG_E_UNSUPPORTED,
                        "decode kernel owns 16-row x 1..32-column "
                        "sub-tensors (partition %d x %d)", cfg.bm, cfg.bn);
        cfg.bm = 16;
        const SkinnyGeo geo = skinny_geo(p, cfg.bn);
        const int64_t progs = (p.N + cfg.bn - 1) / cfg.bn;
        if (cfg.splitk == 0) {
            // split K over programs until there are four programs per
            // compute unit, keeping at least four super-steps per split
            // (one per wavefront of a four-wavefront program), within the
            // caller's workspace.  Measured over the decode shapes (M 1
            // and 8, bf16 and e4m3, cold weights): within 3 % of the best
            // configuration of each shape on average.
            int64_t sk = 1;
            while (!one_round && !resident && sk < 8 &&
                   progs * sk < 4 * ncu &&
                   (geo.supers + 2 * sk - 1) / (2 * sk) >= 4)
                sk *= 2;
            while (sk > 1 &&
                   skinny_ws_bytes(effective_splitk(geo.supers, sk, nullptr),
                                   p.M, p.N, norm) > have)
                sk /= 2;
            cfg.splitk = (int32_t)sk;
        }
        if (cfg.splitk < 1 || cfg.splitk > TG_MAX_SPLITK)
            return fail(TG_E_UNSUPPORTED, "splitk %d not in [1, %d]",
                        cfg.splitk, TG_MAX_SPLITK);
        int64_t per = 1;
        cfg.splitk = effective_splitk(geo.supers, cfg.splitk, &per);
        L.sps = (int32_t)std::min<int64_t>(per * geo.unroll, INT32_MAX);
        if (cfg.ksplit == 0) {
            // four wavefronts per program split K, and at least one
            // wavefront per compute unit.  Measured on the decode shapes
            // with cold weights, where each wavefront keeps two super-steps
            // of loads in flight.
            int ks = 4;
            while (ks < 16 && progs * cfg.splitk * ks < ncu) ks *= 2;
            // one round of programs: eight wavefronts for e4m3 weights
            // (half the bytes per K element; measured 3-9 % faster than
            // four) except with more than four rows over long K ((8, 5120,
            // 25600): four are 5 % faster), four for bf16
            if (one_round && p.b_dt == TG_FP8_E4M3 &&
                !(p.M > 4 && p.K > 8192))
                ks = 8;
            if (resident) ks = 1;
            if (halves) ks = 2;
            // e4m3 weights, one or two activation rows, several programs
            // per compute unit: two wavefronts per 16-column program
            // (measured at (1 and 2, 51200, 5120), (1, 16384, 4096) and
            // (1, 16384, 16384): 6-12 % faster than 32-column programs of
            // four wavefronts; 4 % slower at (1, 32768, 4096))
            if (!one_round && p.b_dt == TG_FP8_E4M3 && p.M <= 2 &&
                cfg.bn == 16 && cfg.splitk == 1 && progs >= ncu)
                ks = 2;
            // no more wavefronts than super-steps of K (eight 16-byte
            // weight loads per lane each) in one split
            while (ks > 1 && ks > per) ks /= 2;
            cfg.ksplit = ks;
        }
        if (cfg.ksplit != 1 && cfg.ksplit != 2 && cfg.ksplit != 4 &&
            cfg.ksplit != 8 && cfg.ksplit != 16)
            return fail(TG_E_UNSUPPORTED, "ksplit %d not in {1,2,4,8,16}",
                        cfg.ksplit);
        // the streaming form (not of the fused normalisation), reported as
        // the stages of its ring
        L.stream = norm || cfg.splitk > 1
                       ? 0
                       : skinny_stream(p.b_dt, p.M, p.N, p.K,
                                       row_stride(*A).ld, row_stride(*B).ld,
                                       cfg.bn, cus);
        cfg.stages = L.stream ? kStreamRing : 0;
        cfg.bk = p.b_dt == TG_BF16 ? 32 : 64;
        cfg.wm = 1;
        cfg.wn = 1;
        L.s.tiles_m = 1;
        L.s.tiles_n = (int32_t)((p.N + cfg.bn - 1) / cfg.bn);
        L.s.n_tiles = L.s.tiles_n;
        L.s.n_prog = L.s.n_tiles;
        L.s.group_m = 1;
        L.gm = L.gn = 1;
    } else if (cfg.kind == TG_KIND_TILED) {
        if (!t_ok)
            return fail(TG_E_UNSUPPORTED,
                        "tiled kernel needs matching A/B dtypes, 16-byte "
                        "aligned rows, K (and N for B stored K x N) a "
                        "multiple of 16 bytes, e4m3 B stored N x K");
        if (cfg.bm == 0 && cfg.bn == 0) {
            if (cfg.wm == 0 && cfg.wn == 0 && cfg.bk == 0 &&
                cfg.stages == 0 && cfg.sched == 0) {
                const DefaultTile t = default_tile(L.gemm_dt, p.M, p.N, L.Kc,
                                                   p.b_nk, cus);
                cfg.bm = cfg.bn = t.size;
                cfg.stages = t.stages;
                cfg.wm = t.wm;
            } else {
                cfg.bm = cfg.bn = named_tile(L.gemm_dt, p.M, p.N, cus);
            }
        } else if (cfg.bm == 0 || cfg.bn == 0) {
            return fail(TG_E_ARG, "config bm/bn: set both or neither");
        }
        if (cfg.bm == 128 && cfg.bn == 128 && cfg.wm == 0 && cfg.wn == 0 &&
            cfg.bk == 0 && cfg.stages == 0 && cfg.sched == 0 &&
            L.gemm_dt != TG_F32)
            cfg.stages = rounds_128(tiles_of(p.M, p.N, 128), cus);
        // Long K (at least 16384 and twice the larger of M and N) keeps its
        // own schedule name, which plans and tuning files carry; the kernel
        // is the phased one either way.
        if (cfg.sched == 0 && cfg.wm == 0 && cfg.wn == 0 && cfg.bk == 0 &&
            cfg.stages == 0 && L.gemm_dt == TG_BF16 && p.b_nk &&
            cfg.bm == 256 && cfg.bn == 256 && L.Kc >= 16384 &&
            L.Kc >= 2 * std::max(p.M, p.N))
            cfg.sched = TG_SCHED_CROSS_WARM;
        L.variant = find_variant(L.gemm_dt, cfg.bm, cfg.bn, cfg.wm, cfg.wn,
                                 cfg.bk, cfg.stages, cfg.sched, p.b_nk,
                                 p.c_bf16, chunk_multiple(L.Kc, L.gemm_dt),
                                 p.scaled, L.Kc % 64 == 0, L.Kc % 32 == 0);
        if (L.variant < 0)
            return fail(TG_E_UNSUPPORTED,
                        "no tiled kernel for dtype %d, %d x %d, waves %d x %d,"
                        " bk %d, %d stages, schedule %d (ping-pong needs K a "
                        "multiple of 16 bytes)", L.gemm_dt, cfg.bm, cfg.bn,
                        cfg.wm, cfg.wn, cfg.bk, cfg.stages, cfg.sched);
        const TiledVariant &v = tiled_variant(L.variant);
        cfg.bk = v.bk;
        cfg.wm = v.wm;
        cfg.wn = v.wn;
        cfg.stages = v.stages;
        cfg.sched = v.sched;
        cfg.ksplit = 1;
        if (cfg.splitk > 1)
            return fail(TG_E_UNSUPPORTED, "splitk applies to the decode "
                                          "kernel only");
        cfg.splitk = 1;
        L.sps = 0;
        L.s.tiles_m = (int32_t)((p.M + cfg.bm - 1) / cfg.bm);
        L.s.tiles_n = (int32_t)((p.N + cfg.bn - 1) / cfg.bn);
        L.s.n_tiles = L.s.tiles_m * L.s.tiles_n;
        int occ = cus > 0 ? tiled_occupancy(L.variant) : 1;
        int64_t cap = (int64_t)(cus > 0 ? cus : 256) * occ;
        // binary32: one program per sub-tensor.  Its matrix instructions take
        // 32 times as long per byte as the bf16 ones, so loads need no
        // stream across sub-tensors, and the dispatcher levels an uneven
        // last round that a fixed deal leaves on two of the eight XCDs.
        L.s.n_prog = L.gemm_dt == TG_F32
                         ? L.s.n_tiles
                         : (int32_t)std::min<int64_t>(L.s.n_tiles, cap);
        L.s.group_m = 8;
    } else {  // simple
        if (np > 1)
            return fail(TG_E_UNSUPPORTED,
                        "split precision runs on the tiled kernel only");
        if (cfg.bm == 0 && cfg.bn == 0) cfg.bm = cfg.bn = 64;
        if (cfg.bm <= 0 || cfg.bn <= 0 || cfg.bm > 64 || cfg.bn > 64)
            return fail(TG_E_UNSUPPORTED,
                        "simple kernel partitions are at most 64 x 64");
        cfg.ksplit = 1;
        if (cfg.splitk > 1)
            return fail(TG_E_UNSUPPORTED, "splitk applies to the decode "
                                          "kernel only");
        cfg.splitk = 1;
        L.sps = 0;
        L.s.tiles_m = (int32_t)((p.M + cfg.bm - 1) / cfg.bm);
        L.s.tiles_n = (int32_t)((p.N + cfg.bn - 1) / cfg.bn);
        L.s.n_tiles = L.s.tiles_m * L.s.tiles_n;
        simple_group(L, cfg, cus);
        L.s.n_prog = simple_blocks_m(L) *
                     ((L.s.tiles_n + L.gn - 1) / L.gn);
        L.s.group_m = 1;
        // K tiles, wavefronts and LDS stages of the kernel that runs
        L.cfg = cfg;
        L.mixed = mixed_ok(p, A, B, C, L);
        cfg.bk = p.a_dt == TG_F32 ? 32 : 64;
        cfg.wm = L.mixed ? 4 : 2;
        cfg.wn = !L.mixed && (L.gm * cfg.bm > 64 || L.gn * cfg.bn > 64) ? 4
                                                                        : 2;
        cfg.stages = L.mixed ? 4 : 2;
    }
    L.cfg = cfg;
    return TG_OK;
}

host::Key key_of(const Problem &p) {
    host::Key k;
    k.M = p.M; k.N = p.N; k.K = p.K;
    k.a_dt = p.a_dt; k.b_dt = p.b_dt; k.b_nk = p.b_nk; k.c_bf16 = p.c_bf16;
    k.precision = p.precision;
    return k;
}

tg_config default_config(const Problem &p, const tg_in *A, const tg_in *B,
                         const tg_out *C);

// Every launch tile_gemm can make for this request, each under one name: the
// heuristic's where that is one of several (the tuner would choose between
// names by noise, and the picker learn differences that are none).
void candidates(const Problem &p, const tg_in *A, const tg_in *B,
                const tg_out *C, std::vector<tg_config> &out) {
    out.clear();
    const tg_config dflt = default_config(p, A, B, C);
    auto try_cfg = [&](const tg_config &c) {
        Launch L;
        std::string keep = g_err;
        tg_status st = choose_explicit(p, A, B, C, &c, L, SIZE_MAX);
        if (st == TG_OK && L.stream) {
            // the streaming form has no use for ksplit: the one that the
            // plain form's rule gives, for calls whose strides need that
            tg_config one = c;
            one.ksplit = dflt.kind == TG_KIND_SKINNY && dflt.bn == c.bn &&
                                 dflt.splitk == 1 ? dflt.ksplit : 0;
            st = choose_explicit(p, A, B, C, &one, L, SIZE_MAX);
        }
        if (st == TG_OK) {
            bool dup = false;
            for (const tg_config &o : out)
                dup = dup || std::memcmp(&o, &L.cfg, sizeof o) == 0;
            if (!dup) out.push_back(L.cfg);
        }
        g_err = keep;
    };
    const int np = p.precision == TG_PREC_BF16X3 ? 3
                   : p.precision == TG_PREC_BF16X6 ? 6 : 1;
    const int gdt = np > 1 ? TG_BF16 : p.a_dt;
    const int cus = device_cus();
    const int32_t bal = balanced_bn(p.N, cus > 0 ? cus : 256);
    // 16- and 32-column programs, and the column count that deals N evenly
    // over the compute units
    for (int bn : {16, 32, bal == 16 || bal == 32 ? 0 : bal})
        for (int sk : {1, 2, 4, 8})
            for (int ks : {1, 2, 4, 8, 16}) {
                // K split over programs with two to eight wavefronts each
                if (bn == 0 || (sk > 1 && (ks < 2 || ks > 8))) continue;
                tg_config c{};
                c.kind = TG_KIND_SKINNY;
                c.bn = bn;
                c.ksplit = ks;
                c.splitk = sk;
                try_cfg(c);
            }
    const int n = tiled_variant_count();
    auto is_default = [&](const TiledVariant &v) {
        return dflt.kind == TG_KIND_TILED && dflt.bm == v.bm &&
               dflt.bn == v.bn && dflt.bk == v.bk && dflt.wm == v.wm &&
               dflt.wn == v.wn && dflt.stages == v.stages &&
               dflt.sched == v.sched;
    };
    for (int i = 0; i < n; ++i) {
        const TiledVariant &v = tiled_variant(i);
        if (v.dtype != gdt || v.b_nk != (int)p.b_nk || v.c_bf16 != (int)p.c_bf16)
            continue;
        bool named = false;    // this kernel is listed under another name
        for (int j = 0; j < n && !is_default(v); ++j)
            named = named || (j != i && tiled_kernel(j) == tiled_kernel(i) &&
                              (j < i || is_default(tiled_variant(j))));
        if (named) continue;
        tg_config c{};
        c.kind = TG_KIND_TILED;
        c.bm = v.bm; c.bn = v.bn; c.wm = v.wm; c.wn = v.wn;
        c.bk = v.bk; c.stages = v.stages; c.sched = v.sched;
        try_cfg(c);
    }
    // the element-wise fallback competes only where nothing else runs
    if (!out.empty()) return;
    for (int t : {64, 32}) {
        tg_config c{};
        c.kind = TG_KIND_SIMPLE;
        c.bm = c.bn = t;
        try_cfg(c);
    }
}

float lg2(double x) { return (float)std::log2(x < 1.0 ? 1.0 : x); }

// Picker features of one (request, configuration) pair.
// dflt: the configuration the fixed heuristic gives the same request; the
// last feature flags the candidate that equals it, so that the model learns
// its corrections relative to the heuristic.
void features(const Problem &p, const Launch &L, const tg_config &dflt,
              float *f) {
    const tg_config &c = L.cfg;
    const double tiles = L.s.n_tiles > 0 ? L.s.n_tiles : 1;
    const double progs = L.s.n_prog > 0 ? L.s.n_prog : 1;
    const double rounds = std::ceil(tiles / progs);
    const auto pos = [](int v) { return (double)(v > 0 ? v : 1); };
    f[0] = lg2((double)p.M);
    f[1] = lg2((double)p.N);
    f[2] = lg2((double)(p.K > 0 ? p.K : 1));
    f[3] = (p.a_dt == TG_FP8_E4M3 || p.b_dt == TG_FP8_E4M3) ? 1.f : 0.f;
    f[4] = p.a_dt == TG_F32 ? 1.f : 0.f;
    f[5] = p.b_nk ? 1.f : 0.f;
    f[6] = p.c_bf16 ? 1.f : 0.f;
    f[7] = c.kind == TG_KIND_TILED ? 1.f : 0.f;
    f[8] = c.kind == TG_KIND_SKINNY ? 1.f : 0.f;
    f[9] = c.kind == TG_KIND_SIMPLE ? 1.f : 0.f;
    f[10] = lg2((double)c.bm);
    f[11] = lg2((double)c.bn);
    f[12] = lg2(pos(c.wm * c.wn));
    f[13] = c.kind == TG_KIND_TILED ? lg2(pos(c.stages)) : 0.f;
    f[14] = lg2(pos(c.ksplit));
    f[15] = lg2(tiles);
    f[16] = lg2(progs);
    f[17] = lg2(rounds);
    f[18] = (float)(tiles / (progs * rounds));
    f[19] = (float)((double)p.M * (double)p.N /
                    (tiles * (double)c.bm * (double)c.bn));
    f[20] = c.sched == TG_SCHED_PINGPONG ? 1.f : 0.f;
    f[21] = c.sched == TG_SCHED_CROSS        ? 1.f
            : c.sched == TG_SCHED_CROSS_WARM ? 2.f
                                             : 0.f;
    f[22] = lg2(pos(c.splitk));
    f[23] = std::memcmp(&c, &dflt, sizeof c) == 0 ? 1.f : 0.f;
}

// The heuristic's configuration for a request (what tile_gemm runs with
// neither cache nor model), given a workspace; zeros when none applies.
tg_config default_config(const Problem &p, const tg_in *A, const tg_in *B,
                         const tg_out *C) {
    Launch L0;
    std::string keep = g_err;
    tg_config d{};
    if (choose_explicit(p, A, B, C, nullptr, L0, SIZE_MAX) == TG_OK)
        d = L0.cfg;
    g_err = keep;
    return d;
}

// Configuration when the caller gives none: the tuning cache, then the
// learned picker's argmin over the candidates, then the fixed heuristic.
// `have`: workspace bytes the caller supplies.  Tuned or predicted
// configurations whose decode split needs more are passed over.
tg_status choose(const Problem &p, const tg_in *A, const tg_in *B,
                 const tg_out *C, const tg_opts *o, Launch &L, size_t have,
                 bool norm = false) {
    const tg_config *uc = o ? o->config : nullptr;
    if (uc || C->bm > 0 || C->bn > 0)
        return choose_explicit(p, A, B, C, uc, L, have, norm);
    const int mode = host::picker_mode();
    tg_config cfg;
    auto fits = [&](const Launch &Lx) {
        return Lx.cfg.kind != TG_KIND_SKINNY ||
               skinny_ws_bytes(Lx.cfg.splitk, p.M, p.N, norm) <= have;
    };
    if ((mode & host::kUseCache) && host::cache_find(key_of(p), &cfg)) {
        if (choose_explicit(p, A, B, C, &cfg, L, have, norm) == TG_OK &&
            fits(L))
            return TG_OK;
    }
    if ((mode & host::kUseMlp) && host::picker_ready()) {
        std::vector<tg_config> cands;
        candidates(p, A, B, C, cands);
        float best = 0.f;
        int bi = -1;
        const tg_config dflt = default_config(p, A, B, C);
        for (size_t i = 0; i < cands.size(); ++i) {
            Launch Li;
            if (choose_explicit(p, A, B, C, &cands[i], Li, have, norm) !=
                    TG_OK ||
                !fits(Li))
                continue;
            float f[TG_PICKER_FEATURES];
            features(p, Li, dflt, f);
            const float y = host::picker_predict(f);
            if (bi < 0 || y < best) {
                best = y;
                bi = (int)i;
            }
        }
        if (bi >= 0)
            return choose_explicit(p, A, B, C, &cands[bi], L, have, norm);
    }
    return choose_explicit(p, A, B, C, nullptr, L, have, norm);
}

// Calls own(p, id) for every sub-tensor id of every program p, in the order
// the kernels walk them; stops where own returns false.
template <class Own>
bool walk_map(const Launch &L, Own own) {
    const Sched &s = L.s;
    for (int32_t p = 0; p < s.n_prog; ++p) {
        if (L.cfg.kind == TG_KIND_SIMPLE) {
            int32_t bm, bn;
            simple_block(p, s.n_prog, simple_blocks_m(L), bm, bn);
            for (int32_t tm = bm * L.gm;
                 tm < std::min((bm + 1) * L.gm, s.tiles_m); ++tm)
                for (int32_t tn = bn * L.gn;
                     tn < std::min((bn + 1) * L.gn, s.tiles_n); ++tn)
                    if (!own(p, tm * s.tiles_n + tn)) return false;
        } else if (L.cfg.kind == TG_KIND_TILED) {
            for (int32_t t = program_slot(p, s.n_prog); t < s.n_tiles;
                 t += s.n_prog) {
                int32_t tm, tn;
                tile_coords(t, s, tm, tn);
                if (!own(p, tm * s.tiles_n + tn)) return false;
            }
        } else if (!own(p, p)) {   // one program per sub-tensor, row-major
            return false;
        }
    }
    return true;
}

// Program p -> owned sub-tensor ids.
void build_map(const Launch &L, int32_t *offs, int32_t *ids) {
    int32_t q = 0;
    std::fill(offs, offs + L.s.n_prog + 1, 0);
    walk_map(L, [&](int32_t p, int32_t id) {
        ids[q++] = id;
        offs[p + 1] = q;
        return true;
    });
    for (int32_t p = 0; p < L.s.n_prog; ++p)
        offs[p + 1] = std::max(offs[p + 1], offs[p]);
}

// The program map a launch will walk, checked with the rules of
// tile_partition_check (injective, covering) as it is walked.
tg_status check_launch_map(const Launch &L) {
    // reused per thread: after the first call of a size, checking
    // allocates nothing
    static thread_local std::vector<uint8_t> seen;
    const int32_t tiles = L.s.n_tiles;
    if (L.s.n_prog == 0) return TG_OK;
    seen.assign((size_t)tiles, 0);
    int32_t owned = 0;
    tg_status st = TG_OK;
    walk_map(L, [&](int32_t p, int32_t t) {
        if (t < 0 || t >= tiles)
            st = fail(TG_E_ARG, "program %d: sub-tensor %d off the grid", p,
                      t);
        else if (seen[(size_t)t])
            st = fail(TG_E_OVERLAP,
                      "sub-tensor %d owned by two programs (second: %d)", t,
                      p);
        else
            seen[(size_t)t] = 1, ++owned;
        return st == TG_OK;
    });
    if (st == TG_OK && owned != tiles)
        return fail(TG_E_NOCOVER, "%d of %d sub-tensors owned by no program",
                    tiles - owned, tiles);
    return st;
}

size_t split_bytes(const Problem &p, int np) {
    return up256((size_t)p.M * p.K * np * 2) +
           up256((size_t)p.K * p.N * np * 2);
}

int planes_of(int precision) {
    return precision == TG_PREC_BF16X3 ? 3
           : precision == TG_PREC_BF16X6 ? 6 : 1;
}

// Plane blocks along the concatenated K axis, smallest products first.
// Entries are (A plane, B plane) with 0 = hi, 1 = mid, 2 = lo.
const int8_t kX3A[3] = {0, 1, 0}, kX3B[3] = {1, 0, 0};
const int8_t kX6A[6] = {1, 2, 0, 1, 0, 0}, kX6B[6] = {1, 0, 2, 0, 1, 0};

// Consistency tag of a grouped plan: a mix of its fields, so that a plan
// prepare did not fill (or one altered since) is refused.
uint64_t plan_tag(const tg_grouped_plan &pl) {
    uint64_t h = 0x9e3779b97f4a7c15ull ^ (uint64_t)(uintptr_t)pl.workspace;
    const int32_t f[4] = {pl.n, pl.total_tiles, pl.n_prog, pl.variant};
    for (int32_t v : f) {
        h ^= (uint64_t)(uint32_t)v + 0x9e3779b97f4a7c15ull + (h << 6) +
             (h >> 2);
        h *= 0xff51afd7ed558ccdull;
    }
    return h;
}

// Device scratch of the allocation-free entry point: one array per device
// (each device holds its own copy at its own address), resolved once per
// device with that device current.  In host code the array's name is
// only a stand-in; the resolved address is the one kernels receive.
__device__ __align__(256) char scratch[TG_NOALLOC_SCRATCH_BYTES];

std::mutex g_scratch_mu;
std::unordered_map<int, void *> g_scratch_addr;

tg_status scratch_address(void **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    auto it = g_scratch_addr.find(dev);
    if (it != g_scratch_addr.end()) {
        *out = it->second;
        return TG_OK;
    }
    void *ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e, "scratch address");
    if (!ptr) return fail(TG_E_HIP, "scratch address is NULL");
    g_scratch_addr[dev] = ptr;
    *out = ptr;
    return TG_OK;
}

// The workspace of a split decode product: present, large and aligned
// enough, and sharing no bytes with the operands or the output.
tg_status check_split_ws(const tg_opts *o, const Problem &p, int splitk,
                         bool norm, const tg_in *ins, int n_in,
                         const tg_out *C) {
    const size_t need = skinny_ws_bytes(splitk, p.M, p.N, norm);
    if (!o || !o->workspace || o->workspace_bytes < need)
        return fail(TG_E_WORKSPACE,
                    "decode product split over %d programs per sub-tensor "
                    "needs a workspace of %zu bytes", splitk, need);
    if (!aligned16(o->workspace))
        return fail(TG_E_WORKSPACE, "workspace must be 16-byte aligned");
    Range rw{(uintptr_t)o->workspace, (uintptr_t)o->workspace + need};
    if (intersect(rw, byte_range(C->data, C->rows, C->cols, C->ld,
                                 esize(C->dtype))))
        return fail(TG_E_ALIAS, "workspace shares bytes with the output");
    for (int i = 0; i < n_in; ++i)
        if (intersect(rw, byte_range(ins[i].data, ins[i].rows, ins[i].cols,
                                     ins[i].ld, esize(ins[i].dtype))))
            return fail(TG_E_ALIAS, "workspace shares bytes with input %d",
                        i);
    return TG_OK;
}

// The residual of a decode product (opts->residual): an M x N bf16 or f32
// row-major device matrix, aligned to its element size.  Fills the kernel
// arguments (res = nullptr without one).
tg_status take_residual(const tg_opts *o, const Problem &p, SkinnyArgs &a) {
    a.res = nullptr;
    a.ldr = 0;
    a.res_bf16 = 0;
    if (!o || !o->residual) return TG_OK;
    const tg_in *r = o->residual;
    tg_status st = check_in(r, "residual");
    if (st != TG_OK) return st;
    if (r->dtype != TG_BF16 && r->dtype != TG_F32)
        return fail(TG_E_DTYPE, "residual must be bf16 or f32");
    if (r->trans || r->rows != p.M || r->cols != p.N)
        return fail(TG_E_SHAPE, "residual must be %lld x %lld, row-major",
                    (long long)p.M, (long long)p.N);
    if ((uintptr_t)r->data % (uintptr_t)esize(r->dtype))
        return fail(TG_E_SHAPE, "residual not aligned to its element size");
    a.res = r->data;
    a.ldr = r->ld;
    a.res_bf16 = r->dtype == TG_BF16;
    return TG_OK;
}

}  // namespace

extern "C" {

const char *tg_status_str(int32_t st) {
    switch (st) {
    case TG_OK: return "TG_OK";
    case TG_E_ARG: return "TG_E_ARG";
    case TG_E_DTYPE: return "TG_E_DTYPE";
    case TG_E_SHAPE: return "TG_E_SHAPE";
    case TG_E_OVERLAP: return "TG_E_OVERLAP";
    case TG_E_NOCOVER: return "TG_E_NOCOVER";
    case TG_E_ALIAS: return "TG_E_ALIAS";
    case TG_E_WORKSPACE: return "TG_E_WORKSPACE";
    case TG_E_UNSUPPORTED: return "TG_E_UNSUPPORTED";
    case TG_E_HIP: return "TG_E_HIP";
    default: return "unknown status";
    }
}

const char *tg_last_error(void) { return g_err.c_str(); }

int32_t tg_device_cus(void) { return device_cus(); }

tg_status tile_partition_check(const tg_in *ins, int32_t n_in,
                               const tg_out *out, int32_t n_prog,
                               const int32_t *prog_offsets,
                               const int32_t *prog_tiles) {
    g_err.clear();
    tg_status st;
    if (n_in < 0 || (n_in > 0 && !ins))
        return fail(TG_E_ARG, "bad input list");
    for (int32_t i = 0; i < n_in; ++i) {
        char name[32];
        snprintf(name, sizeof name, "input %d", i);
        if ((st = check_in(&ins[i], name)) != TG_OK) return st;
    }
    if ((st = check_out(out, true)) != TG_OK) return st;
    int64_t tiles = ((out->rows + out->bm - 1) / out->bm) *
                    ((out->cols + out->bn - 1) / out->bn);
    if ((st = check_map(tiles, n_prog, prog_offsets, prog_tiles)) != TG_OK)
        return st;
    return check_alias(ins, n_in, out);
}

size_t tile_gemm_workspace_size(const tg_in *A, const tg_in *B,
                                const tg_out *C, const tg_opts *o) {
    std::string keep = g_err;
    Problem p;
    if (describe(A, B, C, o, p) != TG_OK) {
        g_err = keep;
        return 0;
    }
    int np = planes_of(p.precision);
    if (np > 1) return split_bytes(p, np);
    Launch L;
    size_t need = 0;
    if (choose(p, A, B, C, o, L, SIZE_MAX) == TG_OK &&
        L.cfg.kind == TG_KIND_SKINNY)
        need = skinny_ws_bytes(L.cfg.splitk, p.M, p.N, false);
    g_err = keep;
    return need;
}

tg_status tile_gemm_plan(const tg_in *A, const tg_in *B, const tg_out *C,
                         const tg_opts *o, tg_config *cfg, int32_t *n_prog,
                         int32_t *prog_offsets, int32_t *prog_tiles) {
    g_err.clear();
    Problem p;
    tg_status st = describe(A, B, C, o, p);
    if (st != TG_OK) return st;
    Launch L;
    // the plan for a caller supplying opts->workspace_bytes of workspace
    if ((st = choose(p, A, B, C, o, L, o ? o->workspace_bytes : 0)) != TG_OK)
        return st;
    if (cfg) *cfg = L.cfg;
    if (n_prog) *n_prog = L.s.n_prog;
    if (prog_offsets && prog_tiles) build_map(L, prog_offsets, prog_tiles);
    return TG_OK;
}

tg_status tile_gemm(const tg_in *A, const tg_in *B, tg_out *C,
                    const tg_opts *o, tg_stream stream) {
    g_err.clear();
    Problem p;
    tg_status st = describe(A, B, C, o, p);
    if (st != TG_OK) return st;
    const tg_in a_row = row_stride(*A), b_row = row_stride(*B);
    A = &a_row;
    B = &b_row;
    Launch L;
    const size_t have = o && o->workspace ? o->workspace_bytes : 0;
    if ((st = choose(p, A, B, C, o, L, have)) != TG_OK) return st;
    const bool residual = o && o->residual;
    if (residual && L.cfg.kind != TG_KIND_SKINNY)
        return fail(TG_E_UNSUPPORTED, "a residual is added by the decode "
                                      "kernel only (M <= 16, W stored N x K)");
    const bool checked = !o || o->checked;
    if (checked) {
        // the program map the kernel will walk must be injective and cover
        // the partition of C, and C may not alias A, B or the residual
        if ((st = check_launch_map(L)) != TG_OK) return st;
        tg_out part = *C;
        part.bm = L.cfg.bm;
        part.bn = L.cfg.bn;
        tg_in ins[3] = {*A, *B, residual ? *o->residual : *A};
        if ((st = check_alias(ins, residual ? 3 : 2, &part)) != TG_OK)
            return st;
    }
    C->bm = L.cfg.bm;
    C->bn = L.cfg.bn;
    if (p.M == 0 || p.N == 0) return TG_OK;
    hipStream_t hs = static_cast<hipStream_t>(stream);
    const float *sa = o ? o->scale_a : nullptr;
    const float *sb = o ? o->scale_b : nullptr;
    int32_t *wc = o ? o->write_count : nullptr;
    hipError_t e = hipSuccess;

    if (L.cfg.kind == TG_KIND_SKINNY) {
        SkinnyArgs a;
        a.x = A->data; a.w = B->data; a.y = C->data;
        a.scale_a = sa; a.scale_w = sb; a.wcount = wc;
        a.ldx = A->ld; a.ldw = B->ld; a.ldy = C->ld;
        a.M = (int32_t)p.M; a.N = (int32_t)p.N; a.K = (int32_t)p.K;
        a.bn = L.cfg.bn;
        a.splitk = L.cfg.splitk;
        a.steps_per_split = L.sps;
        a.part = nullptr;
        a.ssq_part = nullptr;
        if ((st = take_residual(o, p, a)) != TG_OK) return st;
        if (a.splitk > 1) {
            const tg_in ins[3] = {*A, *B, residual ? *o->residual : *A};
            if ((st = check_split_ws(o, p, a.splitk, false, ins,
                                     residual ? 3 : 2, C)) != TG_OK)
                return st;
            a.part = static_cast<float *>(o->workspace);
        }
        e = launch_skinny(p.b_dt, p.c_bf16, L.cfg.bn, L.cfg.ksplit, a,
                          L.stream, hs);
        if (e == hipSuccess && a.splitk > 1)
            e = launch_skinny_merge(p.c_bf16, a, false, 0.f, hs);
        return e == hipSuccess ? TG_OK : hip_fail(e, "decode kernel launch");
    }
    if (L.cfg.kind == TG_KIND_SIMPLE) {
        SimpleArgs a;
        a.a = A->data; a.b = B->data; a.c = C->data;
        a.scale_a = sa; a.scale_b = sb; a.wcount = wc;
        a.lda = A->ld; a.ldb = B->ld; a.ldc = C->ld;
        a.M = (int32_t)p.M; a.N = (int32_t)p.N; a.K = (int32_t)p.K;
        a.a_dtype = p.a_dt; a.b_dtype = p.b_dt; a.c_bf16 = p.c_bf16;
        a.b_nk = p.b_nk; a.bm = L.cfg.bm; a.bn = L.cfg.bn;
        a.gm = L.gm; a.gn = L.gn;
        a.blocks_m = simple_blocks_m(L);
        a.n_prog = L.s.n_prog;
        e = L.mixed ? launch_mixed(a, hs) : launch_simple(a, hs);
        return e == hipSuccess ? TG_OK : hip_fail(e, "simple kernel launch");
    }

    GemmArgs g;
    g.a = A->data; g.b = B->data; g.c = C->data;
    g.scale_a = sa; g.scale_b = sb; g.wcount = wc;
    g.lda = A->ld; g.ldb = B->ld; g.ldc = C->ld;
    g.M = (int32_t)p.M; g.N = (int32_t)p.N; g.K = (int32_t)p.K;
    g.s = L.s;
    int np = planes_of(p.precision);
    if (np > 1) {
        size_t need = split_bytes(p, np);
        if (!o || !o->workspace || o->workspace_bytes < need)
            return fail(TG_E_WORKSPACE, "split precision needs %zu bytes",
                        need);
        if (!aligned16(o->workspace))
            return fail(TG_E_WORKSPACE, "workspace must be 16-byte aligned");
        Range rw{(uintptr_t)o->workspace, (uintptr_t)o->workspace + need};
        Range rc = byte_range(C->data, C->rows, C->cols, C->ld,
                              esize(C->dtype));
        Range ra = byte_range(A->data, A->rows, A->cols, A->ld, 4);
        Range rb = byte_range(B->data, B->rows, B->cols, B->ld, 4);
        if (intersect(rw, rc) || intersect(rw, ra) || intersect(rw, rb))
            return fail(TG_E_ALIAS, "workspace shares bytes with an operand");
        char *ws = static_cast<char *>(o->workspace);
        size_t a_bytes = ((size_t)p.M * p.K * np * 2 + 255) & ~(size_t)255;
        uint32_t oa = 0, ob = 0;
        for (int b = 0; b < np; ++b) {
            oa |= (uint32_t)(np == 3 ? kX3A : kX6A)[b] << (4 * b);
            ob |= (uint32_t)(np == 3 ? kX3B : kX6B)[b] << (4 * b);
        }
        // Where the kernel can step from plane to plane itself (whole K
        // tiles in each) every plane is stored once, else once for each
        // product that reads it.
        const bool once = tiled_planes(L.variant) && p.K > 0 &&
                          p.K % tiled_variant(L.variant).bk == 0;
        if (once) {
            g.kp = (int32_t)p.K;
            g.planes_a = oa;
            g.planes_b = ob;
            oa = ob = 0x210;
        }
        const int blocks = once ? (np == 3 ? 2 : 3) : np;
        const int64_t Kc = p.K * blocks;
        // A' = M x (blocks K): plane block b occupies columns [b K, (b+1) K)
        SplitArgs sa_{}, sb_{};
        sa_.src = static_cast<const float *>(A->data);
        sa_.ld = A->ld;
        sa_.dst = reinterpret_cast<uint16_t *>(ws);
        sa_.rows = (int32_t)p.M;
        sa_.cols = (int32_t)p.K;
        sa_.ldd = Kc;
        sa_.plane_stride = p.K;
        sa_.order = oa;
        sa_.blocks = sb_.blocks = blocks;
        sb_.src = static_cast<const float *>(B->data);
        sb_.ld = B->ld;
        sb_.dst = reinterpret_cast<uint16_t *>(ws + a_bytes);
        sb_.order = ob;
        // B stored N x K -> B' = N x (blocks K); stored K x N -> B' =
        // (blocks K) x N: plane block b is rows [b K, (b+1) K)
        sb_.rows = (int32_t)(p.b_nk ? p.N : p.K);
        sb_.cols = (int32_t)(p.b_nk ? p.K : p.N);
        sb_.ldd = p.b_nk ? Kc : p.N;
        sb_.plane_stride = p.b_nk ? p.K : p.K * p.N;
        e = launch_split(sa_, sb_, hs);
        if (e != hipSuccess) return hip_fail(e, "split launch");
        g.a = sa_.dst; g.b = sb_.dst;
        g.lda = Kc;
        g.ldb = sb_.ldd;
        g.K = (int32_t)(p.K * np);
    }
    e = launch_tiled(L.variant, g, hs);
    return e == hipSuccess ? TG_OK : hip_fail(e, "tiled kernel launch");
}

tg_status tile_gemm_noalloc(const tg_in *A, const tg_in *B, tg_out *C,
                            const tg_opts *o, tg_stream stream) {
    g_err.clear();
    if (o && o->workspace)
        return fail(TG_E_ARG, "the allocation-free call takes no workspace");
    void *ptr = nullptr;
    tg_status st = scratch_address(&ptr);
    if (st != TG_OK) return st;
    tg_opts oo{};
    if (o)
        oo = *o;
    else
        oo.checked = 1;
    oo.workspace = ptr;
    oo.workspace_bytes = TG_NOALLOC_SCRATCH_BYTES;
    st = tile_gemm(A, B, C, &oo, stream);
    if (st == TG_E_WORKSPACE)
        g_err = "the allocation-free call's scratch holds " +
                std::to_string((size_t)TG_NOALLOC_SCRATCH_BYTES) +
                " bytes: " + g_err;
    return st;
}

int32_t tile_gemm_candidates(const tg_in *A, const tg_in *B, const tg_out *C,
                             const tg_opts *o, tg_config *out, int32_t max) {
    g_err.clear();
    Problem p;
    if (describe(A, B, C, o, p) != TG_OK) return -1;
    std::vector<tg_config> c;
    candidates(p, A, B, C, c);
    for (int32_t i = 0; i < (int32_t)c.size() && i < max; ++i) out[i] = c[i];
    return (int32_t)c.size();
}

tg_status tile_picker_features(const tg_in *A, const tg_in *B,
                               const tg_out *C, const tg_config *cfg,
                               float *feat) {
    g_err.clear();
    if (!feat) return fail(TG_E_ARG, "NULL feature buffer");
    Problem p;
    tg_status st = describe(A, B, C, nullptr, p);
    if (st != TG_OK) return st;
    Launch L;
    if ((st = choose_explicit(p, A, B, C, cfg, L, SIZE_MAX)) != TG_OK)
        return st;
    features(p, L, default_config(p, A, B, C), feat);
    return TG_OK;
}

// ----------------------------------------------------------------- grouped

size_t tile_gemm_grouped_workspace_size(int32_t n) {
    if (n <= 0) return 0;
    return sizeof(GroupProblem) * (size_t)n;
}

tg_status tile_gemm_grouped_prepare(int32_t n, const tg_in *A,
                                    const tg_in *B, tg_out *C,
                                    const tg_opts *o, void *ws,
                                    size_t ws_bytes, tg_grouped_plan *plan,
                                    tg_stream stream) {
    g_err.clear();
    if (!plan) return fail(TG_E_ARG, "NULL plan");
    if (n <= 0 || !A || !B || !C) return fail(TG_E_ARG, "empty problem list");
    if (!ws) return fail(TG_E_WORKSPACE, "NULL workspace");
    if (ws_bytes < tile_gemm_grouped_workspace_size(n))
        return fail(TG_E_WORKSPACE, "workspace needs %zu bytes",
                    tile_gemm_grouped_workspace_size(n));
    if (!aligned16(ws)) return fail(TG_E_WORKSPACE, "workspace misaligned");
    if (o && (o->precision != TG_PREC_NATIVE || o->scale_a || o->scale_b))
        return fail(TG_E_UNSUPPORTED,
                    "grouped launch: native precision, no scales");
    int32_t *wc = o ? o->write_count : nullptr;
    std::vector<Problem> ps((size_t)n);
    int c_bf16 = -1, b_nk = -1;
    int64_t maxM = 0, maxN = 0;
    for (int32_t i = 0; i < n; ++i) {
        tg_status st = describe(&A[i], &B[i], &C[i], nullptr, ps[i]);
        if (st != TG_OK) {
            g_err = "problem " + std::to_string(i) + ": " + g_err;
            return st;
        }
        if (ps[i].a_dt != TG_BF16 || ps[i].b_dt != TG_BF16)
            return fail(TG_E_DTYPE, "problem %d: grouped launch is bf16", i);
        if (!tiled_ok(ps[i], &A[i], &B[i], &C[i], TG_BF16))
            return fail(TG_E_UNSUPPORTED, "problem %d: layout not tileable",
                        i);
        if (c_bf16 < 0) c_bf16 = ps[i].c_bf16;
        if (b_nk < 0) b_nk = ps[i].b_nk;
        if (c_bf16 != (int)ps[i].c_bf16 || b_nk != (int)ps[i].b_nk)
            return fail(TG_E_UNSUPPORTED,
                        "problem %d: all problems share C dtype and B layout",
                        i);
        maxM = std::max(maxM, ps[i].M);
        maxN = std::max(maxN, ps[i].N);
    }
    // ownership across the launch: outputs pairwise disjoint and disjoint
    // from every input
    std::vector<Range> outs((size_t)n), ins((size_t)2 * n);
    for (int32_t i = 0; i < n; ++i) {
        outs[i] = byte_range(C[i].data, C[i].rows, C[i].cols, C[i].ld,
                             esize(C[i].dtype));
        ins[2 * i] = byte_range(A[i].data, A[i].rows, A[i].cols, A[i].ld, 2);
        ins[2 * i + 1] =
            byte_range(B[i].data, B[i].rows, B[i].cols, B[i].ld, 2);
    }
    for (int32_t i = 0; i < n; ++i) {
        for (int32_t j = i + 1; j < n; ++j)
            if (intersect(outs[i], outs[j]))
                return fail(TG_E_OVERLAP, "outputs %d and %d share bytes", i,
                            j);
        for (int32_t j = 0; j < 2 * n; ++j)
            if (intersect(outs[i], ins[j]))
                return fail(TG_E_ALIAS, "output %d shares bytes with an input "
                                        "of problem %d", i, j / 2);
    }
    // one tile shape for the launch
    tg_config cfg{};
    if (o && o->config) cfg = *o->config;
    if (cfg.bm == 0 || cfg.bn == 0) {
        int64_t work = 0;
        for (auto &p : ps) work += p.M * p.N;
        cfg.bm = cfg.bn = work >= (int64_t)256 * 256 * 256 ? 256 : 128;
    }
    const int cus = device_cus();
    if (cfg.bm == 128 && cfg.bn == 128 && cfg.wm == 0 && cfg.wn == 0 &&
        cfg.bk == 0 && cfg.stages == 0 && cfg.sched == 0) {
        int64_t tiles = 0, longest = 0, sum = 0;
        for (auto &p : ps) {
            const int64_t t = tiles_of(p.M, p.N, 128);
            tiles += t;
            sum += t * p.K;
            if (t > 0) longest = std::max(longest, p.K);
        }
        cfg.stages = grouped_stages_128(tiles, longest, sum, b_nk == 1, cus);
    }
    bool pp_ok = true, tiles_ok = true, k32_ok = true;
    for (auto &p : ps) {
        pp_ok = pp_ok && chunk_multiple(p.K, TG_BF16);
        tiles_ok = tiles_ok && p.K % 64 == 0;
        k32_ok = k32_ok && p.K % 32 == 0;
    }
    int variant = find_variant(TG_BF16, cfg.bm, cfg.bn, cfg.wm, cfg.wn,
                               cfg.bk, cfg.stages, cfg.sched, b_nk == 1,
                               c_bf16 == 1, pp_ok, false, tiles_ok, k32_ok);
    if (variant < 0)
        return fail(TG_E_UNSUPPORTED, "no tiled kernel %d x %d", cfg.bm,
                    cfg.bn);
    for (int32_t i = 0; i < n; ++i) {
        C[i].bm = cfg.bm;
        C[i].bn = cfg.bn;
    }
    // longest K first: programs take tiles in table order with a fixed
    // stride (every other row of them backwards), so the costliest tiles are
    // spread over all programs first
    std::vector<int32_t> order((size_t)n);
    for (int32_t i = 0; i < n; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) {
        return ps[x].K > ps[y].K;
    });
    // problem i's write counters follow those of problems 0 .. i-1
    std::vector<int64_t> wc_off((size_t)n + 1, 0);
    for (int32_t i = 0; i < n; ++i)
        wc_off[i + 1] = wc_off[i] + ps[i].M * ps[i].N;
    std::vector<GroupProblem> tab((size_t)n);
    int64_t total = 0;
    for (int32_t r = 0; r < n; ++r) {
        int32_t i = order[r];
        GroupProblem &g = tab[r];
        g.a = A[i].data; g.b = B[i].data; g.c = C[i].data;
        g.lda = row_stride(A[i]).ld; g.ldb = row_stride(B[i]).ld;
        g.ldc = C[i].ld;
        g.M = (int32_t)ps[i].M; g.N = (int32_t)ps[i].N; g.K = (int32_t)ps[i].K;
        g.tiles_m = (int32_t)((ps[i].M + cfg.bm - 1) / cfg.bm);
        g.tiles_n = (int32_t)((ps[i].N + cfg.bn - 1) / cfg.bn);
        g.tile_begin = (int32_t)total;
        g.c_bf16 = c_bf16;
        g.b_nk = b_nk;
        g.wcount = wc ? wc + wc_off[i] : nullptr;
        total += (int64_t)g.tiles_m * g.tiles_n;
    }
    if (total > INT32_MAX) return fail(TG_E_SHAPE, "too many sub-tensors");
    tg_grouped_plan pl{};
    pl.workspace = ws;
    pl.n = n;
    pl.total_tiles = (int32_t)total;
    int occ = cus > 0 ? tiled_occupancy(variant) : 1;
    pl.n_prog = (int32_t)std::min<int64_t>(total,
                                           (int64_t)(cus > 0 ? cus : 256) * occ);
    if (pl.n_prog < 1) pl.n_prog = 1;
    pl.variant = variant;
    pl.tag = plan_tag(pl);
    hipStream_t hs = static_cast<hipStream_t>(stream);
    hipError_t e = hipMemcpyAsync(ws, tab.data(), sizeof(GroupProblem) * n,
                                  hipMemcpyHostToDevice, hs);
    if (e != hipSuccess) return hip_fail(e, "grouped table copy");
    // the table lives in host memory owned by this call
    e = hipStreamSynchronize(hs);
    if (e != hipSuccess) return hip_fail(e, "grouped table copy");
    *plan = pl;
    return TG_OK;
}

tg_status tile_gemm_grouped(const tg_grouped_plan *plan, tg_stream stream) {
    g_err.clear();
    if (!plan) return fail(TG_E_ARG, "NULL plan");
    if (!plan->workspace || plan->tag != plan_tag(*plan) ||
        plan->variant < 0 || plan->variant >= tiled_variant_count() ||
        plan->n <= 0 || plan->total_tiles < 0 || plan->n_prog < 1)
        return fail(TG_E_ARG,
                    "plan was not filled by tile_gemm_grouped_prepare");
    if (plan->total_tiles == 0) return TG_OK;
    hipError_t e = launch_grouped(plan->variant, plan->n, plan->total_tiles,
                                  plan->n_prog, plan->workspace,
                                  static_cast<hipStream_t>(stream));
    return e == hipSuccess ? TG_OK : hip_fail(e, "grouped kernel launch");
}

tg_status tile_rms_norm_matvec(const tg_in *x, const tg_in *nw, float eps,
                               const tg_in *W, tg_out *y, const tg_opts *o,
                               tg_stream stream) {
    g_err.clear();
    tg_status st;
    if ((st = check_in(nw, "nw")) != TG_OK) return st;
    if (nw->dtype != TG_BF16 || nw->trans || nw->rows != 1)
        return fail(TG_E_SHAPE, "nw must be a 1 x K bf16 row");
    if (!(eps >= 0.0f) || !std::isfinite(eps))
        return fail(TG_E_ARG, "eps must be finite and >= 0");
    if (o && (o->precision != TG_PREC_NATIVE || o->config))
        return fail(TG_E_ARG, "the fused product takes no precision or "
                              "configuration options");
    tg_opts oo{};
    if (o) oo = *o;
    else oo.checked = 1;
    tg_config cfg{};
    cfg.kind = TG_KIND_SKINNY;
    cfg.ksplit = 4;
    oo.config = &cfg;
    const size_t have = o && o->workspace ? o->workspace_bytes : 0;
    Problem p;
    if ((st = describe(x, W, y, &oo, p)) != TG_OK) return st;
    if (nw->cols != p.K)
        return fail(TG_E_SHAPE, "nw has %lld columns, K = %lld",
                    (long long)nw->cols, (long long)p.K);
    if (p.K > 0 && ((uintptr_t)nw->data & 15) != 0)
        return fail(TG_E_SHAPE, "nw must be 16-byte aligned");
    Launch L;
    if ((st = choose(p, x, W, y, &oo, L, have, true)) != TG_OK) return st;
    const bool residual = oo.residual != nullptr;
    if (oo.checked) {
        if ((st = check_launch_map(L)) != TG_OK) return st;
        tg_out part = *y;
        part.bm = L.cfg.bm;
        part.bn = L.cfg.bn;
        tg_in ins[4] = {*x, *W, *nw, residual ? *oo.residual : *x};
        if ((st = check_alias(ins, residual ? 4 : 3, &part)) != TG_OK)
            return st;
    }
    y->bm = L.cfg.bm;
    y->bn = L.cfg.bn;
    if (p.M == 0 || p.N == 0) return TG_OK;
    SkinnyNormArgs a;
    a.s.x = x->data; a.s.w = W->data; a.s.y = y->data;
    a.s.scale_a = oo.scale_a; a.s.scale_w = oo.scale_b;
    a.s.wcount = oo.write_count;
    a.s.ldx = x->ld; a.s.ldw = W->ld; a.s.ldy = y->ld;
    a.s.M = (int32_t)p.M; a.s.N = (int32_t)p.N; a.s.K = (int32_t)p.K;
    a.s.bn = L.cfg.bn;
    a.s.splitk = L.cfg.splitk;
    a.s.steps_per_split = L.sps;
    a.s.part = nullptr;
    a.s.ssq_part = nullptr;
    a.norm_w = nw->data;
    a.eps = eps;
    if ((st = take_residual(&oo, p, a.s)) != TG_OK) return st;
    if (a.s.splitk > 1) {
        const tg_in ins[4] = {*x, *W, *nw, residual ? *oo.residual : *x};
        if ((st = check_split_ws(&oo, p, a.s.splitk, true, ins,
                                 residual ? 4 : 3, y)) != TG_OK)
            return st;
        char *ws = static_cast<char *>(oo.workspace);
        a.s.part = reinterpret_cast<float *>(ws);
        a.s.ssq_part = reinterpret_cast<float *>(
            ws + up256((size_t)a.s.splitk * p.M * p.N * 4));
    }
    hipStream_t hs = static_cast<hipStream_t>(stream);
    hipError_t e = launch_skinny_norm(p.b_dt, p.c_bf16, L.cfg.bn,
                                      L.cfg.ksplit, a, hs);
    if (e == hipSuccess && a.s.splitk > 1)
        e = launch_skinny_merge(p.c_bf16, a.s, true, eps, hs);
    return e == hipSuccess ? TG_OK : hip_fail(e, "fused decode launch");
}

size_t tile_rms_norm_matvec_workspace_size(const tg_in *x, const tg_in *W,
                                           const tg_out *y) {
    std::string keep = g_err;
    tg_config cfg{};
    cfg.kind = TG_KIND_SKINNY;
    cfg.ksplit = 4;
    tg_opts oo{};
    oo.config = &cfg;
    Problem p;
    Launch L;
    size_t need = 0;
    if (describe(x, W, y, &oo, p) == TG_OK &&
        choose(p, x, W, y, &oo, L, SIZE_MAX, true) == TG_OK)
        need = skinny_ws_bytes(L.cfg.splitk, p.M, p.N, true);
    g_err = keep;
    return need;
}

namespace {
tg_status tile_elementwise(bool mul, const tg_in *x, const tg_in *y,
                           tg_out *z, const tg_opts *opts, tg_stream stream) {
    g_err.clear();
    tg_status st;
    if ((st = check_in(x, "x")) != TG_OK) return st;
    if ((st = check_in(y, "y")) != TG_OK) return st;
    if ((st = check_out(z, false)) != TG_OK) return st;
    if (x->trans || y->trans)
        return fail(TG_E_SHAPE, "element-wise operands are not transposed");
    if (x->dtype != z->dtype || y->dtype != z->dtype)
        return fail(TG_E_DTYPE, "x, y and z must share one dtype");
    if (x->rows != z->rows || x->cols != z->cols || y->rows != z->rows ||
        y->cols != z->cols)
        return fail(TG_E_SHAPE, "x, y and z must have one shape");
    const int es = esize(z->dtype), epc = 16 / es;
    if (z->bm == 0 && z->bn == 0) {
        // one row segment of up to 65536 elements per sub-tensor
        z->bm = 1;
        const int64_t bn = std::min<int64_t>(std::max<int64_t>(z->cols, 1),
                                             65536);
        z->bn = (int32_t)((bn + epc - 1) / epc * epc);
    }
    const bool checked = !opts || opts->checked;
    if (checked) {
        const tg_in ins[2] = {*x, *y};
        if ((st = tile_partition_check(ins, 2, z, 0, nullptr, nullptr)) !=
            TG_OK)
            return st;
    } else if (z->bm <= 0 || z->bn <= 0) {
        return fail(TG_E_ARG, "z: partition %d x %d must be positive", z->bm,
                    z->bn);
    }
    if (z->rows == 0 || z->cols == 0) return TG_OK;
    auto al = [](const void *p) { return ((uintptr_t)p & 15) == 0; };
    const bool vec = al(x->data) && al(y->data) && al(z->data) &&
                     (x->ld * es) % 16 == 0 && (y->ld * es) % 16 == 0 &&
                     (z->ld * es) % 16 == 0 && z->bn % epc == 0;
    AddArgs a;
    a.x = x->data; a.y = y->data; a.z = z->data;
    a.wcount = opts ? opts->write_count : nullptr;
    a.ldx = x->rows > 1 ? x->ld : x->cols;
    a.ldy = y->rows > 1 ? y->ld : y->cols;
    a.ldz = z->rows > 1 ? z->ld : z->cols;
    a.rows = z->rows; a.cols = z->cols;
    a.bm = z->bm; a.bn = z->bn;
    a.dtype = z->dtype;
    const int64_t tiles = ((z->rows + z->bm - 1) / z->bm) *
                          ((z->cols + z->bn - 1) / z->bn);
    const int cus = device_cus();
    // sixteen 256-thread programs per compute unit at most (measured at
    // 2^28 bf16 elements: 4 % ahead of four per unit)
    const int programs =
        (int)std::min<int64_t>(tiles, (int64_t)std::max(cus, 1) * 16);
    hipError_t e = (mul ? launch_mul : launch_add)(
        a, vec, programs, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? TG_OK : hip_fail(e, "element-wise launch");
}
}  // namespace

tg_status tile_add(const tg_in *x, const tg_in *y, tg_out *z,
                   const tg_opts *opts, tg_stream stream) {
    return tile_elementwise(false, x, y, z, opts, stream);
}

tg_status tile_mul(const tg_in *x, const tg_in *y, tg_out *z,
                   const tg_opts *opts, tg_stream stream) {
    return tile_elementwise(true, x, y, z, opts, stream);
}

tg_status tile_rms_norm(const tg_in *x, const tg_in *w, float eps,
                        tg_out *y, const tg_opts *opts, tg_stream stream) {
    g_err.clear();
    tg_status st;
    if ((st = check_in(x, "x")) != TG_OK) return st;
    if ((st = check_in(w, "w")) != TG_OK) return st;
    if ((st = check_out(y, false)) != TG_OK) return st;
    if (x->trans || w->trans)
        return fail(TG_E_SHAPE, "normalisation operands are not transposed");
    if (x->dtype != y->dtype || w->dtype != y->dtype)
        return fail(TG_E_DTYPE, "x, w and y must share one dtype");
    if (x->rows != y->rows || x->cols != y->cols)
        return fail(TG_E_SHAPE, "x and y must have one shape");
    if (w->rows != 1 || w->cols != y->cols)
        return fail(TG_E_SHAPE, "w must be 1 x %lld", (long long)y->cols);
    if (!(eps >= 0.0f) || !std::isfinite(eps))
        return fail(TG_E_ARG, "eps must be finite and >= 0");
    if (y->bm == 0 && y->bn == 0) {
        y->bm = 1;
        y->bn = (int32_t)std::max<int64_t>(y->cols, 1);
    }
    if (y->cols > 0 && y->bn != y->cols)
        return fail(TG_E_ARG, "y: sub-tensors must span whole rows (bn %d, "
                    "cols %lld)", y->bn, (long long)y->cols);
    const bool checked = !opts || opts->checked;
    if (checked) {
        const tg_in ins[2] = {*x, *w};
        if ((st = tile_partition_check(ins, 2, y, 0, nullptr, nullptr)) !=
            TG_OK)
            return st;
    } else if (y->bm <= 0 || y->bn <= 0) {
        return fail(TG_E_ARG, "y: partition %d x %d must be positive", y->bm,
                    y->bn);
    }
    if (y->rows == 0 || y->cols == 0) return TG_OK;
    NormArgs a;
    a.x = x->data; a.w = w->data; a.y = y->data;
    a.wcount = opts ? opts->write_count : nullptr;
    a.ldx = x->rows > 1 ? x->ld : x->cols;
    a.ldy = y->rows > 1 ? y->ld : y->cols;
    a.rows = y->rows; a.cols = y->cols;
    a.bm = y->bm;
    a.eps = eps;
    a.dtype = y->dtype;
    const int64_t tiles = (y->rows + y->bm - 1) / y->bm;
    const int programs = (int)std::min<int64_t>(
        tiles, (int64_t)std::max(device_cus(), 1) * 8);
    const int es = esize(y->dtype);
    auto al = [](const void *p) { return ((uintptr_t)p & 15) == 0; };
    const bool vec = al(x->data) && al(w->data) && al(y->data) &&
                     (a.ldx * es) % 16 == 0 && (a.ldy * es) % 16 == 0;
    hipError_t e = launch_rms_norm(a, vec, programs,
                                   static_cast<hipStream_t>(stream));
    return e == hipSuccess ? TG_OK : hip_fail(e, "normalisation launch");
}

tg_status tile_error_norm(const void *C, int32_t c_dtype, const double *R,
                          int64_t n, double *out, tg_stream stream) {
    g_err.clear();
    if (c_dtype != TG_F32 && c_dtype != TG_BF16)
        return fail(TG_E_DTYPE, "C must be TG_F32 or TG_BF16");
    if (n < 0) return fail(TG_E_ARG, "negative n");
    if (!out || (n > 0 && (!C || !R))) return fail(TG_E_ARG, "NULL pointer");
    hipError_t e = launch_error_norm(C, c_dtype == TG_BF16, R, n, out,
                                     static_cast<hipStream_t>(stream));
    return e == hipSuccess ? TG_OK : hip_fail(e, "error-norm launch");
}

}  // extern "C"
