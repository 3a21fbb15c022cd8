// Device kernels (gfx950).  One workgroup transforms one residue row ("limb")
// that stays in LDS for the whole transform; everything else is pointwise.
#pragma once
#include <hip/hip_runtime.h>
#include "tables.hpp"

namespace cg {

// ---------------------------------------------------------------------------
// Transform plan.  A row of N = 2^LOGN residues is transformed by one workgroup
// of N / E threads; each thread keeps E elements in registers and a pass runs
// R butterfly stages on them between two LDS exchanges.  The first NC passes pair
// elements owned by different waves (workgroup barrier); after them every wave
// owns one contiguous chunk of 64 * E elements and all remaining stages stay
// inside it, so those passes only need wave-level ordering.
//   N = 8192: forward kernels run E = 16 (512 threads, registers capped at 128 so that two
//   workgroups share a compute unit and cover each other's loads; no register prefetch), which
//   measured 5-10 % faster than E = 8; the inverse kernels keep E = 8 (their fused loaders spill
//   at 128 registers).  E = 16 is the only choice at N = 16384 (1024 threads).
//   Products at N = 16384 work on half rows: the first stage, which pairs coefficients N / 2 apart, is taken by
//   lift_kernel, which has both in registers, its inverse by scale_kernel, and the two halves of a row are
//   transforms of 8192 with tables of their own (row 2 r + h of prime r).
// ---------------------------------------------------------------------------
template <int LOGN, int E> struct Plan;
template <> struct Plan<14, 16> { static constexpr int NP = 4, NC = 1; static constexpr int R[5] = {4, 4, 3, 3, 0}; };
template <> struct Plan<10, 8> { static constexpr int NP = 4, NC = 1; static constexpr int R[5] = {3, 3, 3, 1, 0}; };      // (parts of rows)
template <> struct Plan<11, 8> { static constexpr int NP = 4, NC = 1; static constexpr int R[5] = {3, 3, 3, 2, 0}; };
template <> struct Plan<12, 8> { static constexpr int NP = 4, NC = 1; static constexpr int R[5] = {3, 3, 3, 3, 0}; };
template <> struct Plan<13, 8> { static constexpr int NP = 5, NC = 2; static constexpr int R[5] = {3, 3, 3, 3, 1}; };
template <> struct Plan<13, 16> { static constexpr int NP = 4, NC = 1; static constexpr int R[5] = {4, 3, 3, 3, 0}; };
// The next row is prefetched into registers where that helps: not with two workgroups on a compute
// unit (each covers the other's load latency), and not at N = 16384, where the prefetched words
// push the 128-register budget of a 1024-thread workgroup into spilling (measured: C5 step
// 4.58 -> 4.29 ms without).
template <int LOGN, int E> constexpr bool prefetch_rows() { return LOGN <= 12 || (LOGN == 13 && E == 8); }
// waves per SIMD the register allocation must leave room for: the workgroup's own, or, for rows of
// 8192 on 512 threads, twice that, so that two workgroups share a compute unit (2 x 72 KiB of LDS)
template <int LOGN, int E> constexpr int min_waves() { return (LOGN == 13 && E == 16) ? 4 : ((1 << LOGN) / E) / 256; }

constexpr int ilog2c(int x) { return x <= 1 ? 0 : 1 + ilog2c(x / 2); }
template <int E> constexpr int chunk_log() { return 6 + ilog2c(E); }

template <int LOGN, int E, int PASS> constexpr int stage_start()
{
    int s = 0;
    for (int i = 0; i < PASS; i++) s += Plan<LOGN, E>::R[i];
    return s;
}

// group index of a thread in pass PASS (g-th group of the thread)
template <int LOGN, int E, int PASS> __device__ __forceinline__ int group_index(int tid, int g)
{
    constexpr int R = Plan<LOGN, E>::R[PASS];
    if (PASS < Plan<LOGN, E>::NC) return tid + g * ((1 << LOGN) / E);
    // Wave-local passes are free in which groups a lane takes.  pad() gives the index bits 0 ... 8 the
    // weights 1, 2, 4, 8, 16, 2, 4, 8, 16 modulo the 32 doubles that 32 lanes read at once (16 lanes write at
    // once, and 16 lanes read or write 16 bytes each): lanes are put on index bits of different weights.
    constexpr int L = LOGN - stage_start<LOGN, E, PASS>() - R;
    const int lane = tid & 63;
    int q = lane;
    if (L == 4 && R == 3) q = (lane & 15) | ((lane & 16) << 1) | ((lane & 32) >> 1);                  // bits 0-3, 8, 7
    if (L == 1 && R == 3) q = (lane & 33) | ((lane & 14) << 1) | ((lane & 16) >> 3);                  // bits 0, 5, 6, 7, 4, 8
    if (L == 3 && R == 3) q = (lane & 7) | ((lane & 24) << 1) | ((lane & 32) >> 2);                   // bits 0-2, 7, 8, 6
    if (L == 0 && R == 3) q = ((lane & 3) << 2) | ((lane & 12) >> 2) | (lane & 48);                   // bits 5, 6, 3, 4, 7, 8
    return ((tid >> 6) << (chunk_log<E>() - R)) + q + 64 * g;
}
// Workgroup barrier that orders LDS traffic only.  __syncthreads() also waits for every
// outstanding global load (vmcnt(0)), which would drain the next row's prefetch at each
// barrier; threads of these kernels exchange data through LDS alone.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
// compiler-level ordering between LDS writes and reads of the same wave (the LDS pipeline
// itself executes one wave's operations in order)
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
}

// Forward stage bound: |out| <= 1.1875 |in| + 0.5 (in units of p).  Values must
// stay below 8p = 2^53.
constexpr double fwd_grow(double b, int stages)
{
    for (int i = 0; i < stages; i++) b = 1.1875 * b + 0.5;
    return b;
}
// Decide at compile time which forward passes start with a reduction.  Only the operands that are not
// multiplied in the first stage (half of them) need it: a product of an operand below 8p is below 2p
// anyway, |out| <= (0.51 + 0.5 + 0.1875 |in|) p after that stage.
// (Bounds are in units of 2^50, above every prime: a product's quotient is off by 3/16 at most per 2^50
// of the lazy operand whatever the prime, so they hold for primes of different sizes too.)
constexpr double FWD_IN = 1.25;      // what loaders deliver
constexpr double LAZY_MAX = 7.9;     // values must stay below 2^53
// IN: bound of the transform's input, in hundredths
template <int LOGN, int E, int PASS, int IN = (int)(100 * FWD_IN)> struct FwdBound {
    static constexpr double in = FwdBound<LOGN, E, PASS - 1, IN>::out;
    static constexpr bool reduce = fwd_grow(in, Plan<LOGN, E>::R[PASS]) > LAZY_MAX;
    static constexpr double out = reduce ? fwd_grow(1.01 + 0.1875 * in, Plan<LOGN, E>::R[PASS] - 1)
                                         : fwd_grow(in, Plan<LOGN, E>::R[PASS]);
};
template <int LOGN, int E, int IN> struct FwdBound<LOGN, E, 0, IN> {
    static constexpr bool reduce = false;
    static constexpr double out = fwd_grow(0.01 * IN, Plan<LOGN, E>::R[0]);
};

// Inverse passes: a sum is as large as its operands together, a product (a - b) w at most
// 0.5 + 0.1875 |a - b|.  The plan of a pass, from the bound of its inputs: which operands are reduced
// before a stage (their sum would pass LAZY_MAX) and which results are reduced at its end, so that the
// next pass starts from INV_OUT.  Of eight results of a three-stage pass two or three are reduced, and
// two operands on the way, where reducing every input takes eight.
// last: the stage that ends the transform, 1 with N^-1 folded into both of its products, 2 without: its sums stay below last_max.
constexpr double INV_OUT = 1.92;
template <int R> struct InvPlan {
    bool before[R][1 << R], after[1 << R];
    double out;
    int reds;
};
// both: of two operands whose sum is too large both are reduced, else the larger one alone where that is enough
template <int R> constexpr InvPlan<R> inv_plan(double in, int last, double last_max, bool both)
{
    InvPlan<R> P{};
    double b[1 << R] = {};
    for (int c = 0; c < (1 << R); c++) b[c] = in;
    for (int s = 0; s < R; s++) {
        const int half = 1 << s;
        const double max = last == 2 && s == R - 1 ? last_max : LAZY_MAX;
        for (int c = 0; c < (1 << R); c++) {
            if (c & half) continue;
            if (b[c] + b[c + half] > max) {
                const bool low = b[c] > b[c + half], one = !both && (low ? b[c + half] : b[c]) + 0.51 <= max;
                for (int i : {c, c + half}) {
                    P.before[s][i] = b[i] > 0.51 && (!one || (i == c) == low);
                    if (P.before[s][i]) {
                        b[i] = 0.51;
                        P.reds++;
                    }
                }
            }
            const double sum = b[c] + b[c + half], prod = 0.5 + 0.1875 * sum;
            b[c] = (last == 1 && s == R - 1) ? prod : sum;
            b[c + half] = prod;
        }
    }
    for (int c = 0; c < (1 << R); c++) {
        P.after[c] = !last && b[c] > INV_OUT;
        if (P.after[c]) {
            b[c] = 0.51;
            P.reds++;
        }
        if (b[c] > P.out) P.out = b[c];
    }
    return P;
}
template <int R> constexpr InvPlan<R> inv_plan(double in, int last, double last_max)
{
    const InvPlan<R> two = inv_plan<R>(in, last, last_max, true), one = inv_plan<R>(in, last, last_max, false);
    return one.reds < two.reds ? one : two;
}
// IN: bound of what the loader delivers, in hundredths; 0: the first pass (NP - 1) reduces it
template <int LOGN, int E, int PASS, int IN, bool FIRST = PASS == Plan<LOGN, E>::NP - 1> struct InvBound {
    static constexpr double in = inv_plan<Plan<LOGN, E>::R[PASS + 1]>(InvBound<LOGN, E, PASS + 1, IN>::in, 0, 0.0).out;
};
template <int LOGN, int E, int PASS, int IN> struct InvBound<LOGN, E, PASS, IN, true> {
    static constexpr double in = IN ? 0.01 * IN : 0.51;
};
// Products of transformed rows: the first factor reduced, the second as a forward transform (of whatever width, in parts or not) leaves it
constexpr int hundredths(double x) { return (int)(100.0 * x) + 1; }
template <int LOGN, int E, int IN> constexpr double fwd_end() { return FwdBound<LOGN, E, Plan<LOGN, E>::NP - 1, IN>::out; }
template <int LOGN> constexpr double fwd_out()
{
    constexpr int in = (int)(100 * FWD_IN), in1 = hundredths(fwd_grow(FWD_IN, 1)), in2 = hundredths(fwd_grow(FWD_IN, 2));
    const double ends[] = {fwd_end<LOGN, 8, in>(), fwd_end<LOGN, LOGN == 13 ? 16 : 8, in>(), fwd_end<LOGN - 1, 8, in1>(), fwd_end<LOGN - 2, 8, in2>()};
    double most = 0.0;
    for (double e : ends) most = e > most ? e : most;
    return most;
}
constexpr double prod_of(double lazy) { return 0.5 + 0.375 * 0.51 * lazy; }

__device__ __forceinline__ void bfly_fwd(double &a, double &b, double w, const ModD m)
{
    const double t = mulmod(b, w, m);
    b = a - t;
    a = a + t;
}
__device__ __forceinline__ void bfly_inv(double &a, double &b, double w, const ModD m)
{
    const double d = a - b;
    a = a + b;
    b = mulmod(d, w, m);
}

// ---------------------------------------------------------------------------
// twiddles of one pass, fetched into registers ahead of the synchronisation
// that precedes the pass: slot (g, (1<<u) - 1 + j) holds the factor of stage
// S0+u for the j-th sub-block of group g
// ---------------------------------------------------------------------------
constexpr int TWREGS = 16;

// LDS layout: two pad doubles after every 32.  What a compute unit's LDS does (probe with 1024-thread workgroups, clocks
// at 2.4 GHz per wave instruction): ds_read_b64 2.4 when 32 lanes hit 32 different doubles modulo 32, 4.3 with two
// of them on one; ds_write_b64 6.6 when 16 lanes hit different doubles modulo 16, 8.1 otherwise; ds_read_b128 4.3,
// ds_write_b128 14.  With this layout and the lanes of group_index the butterfly passes are free of conflicts on paper and
// neighbouring pairs stay 16-byte aligned; the counters show 0.3 to 2 % of LDS cycles lost where 6 to 11 % were with one pad
// after every 8 (what is left is highest in the kernels that permute by a Galois map, 3 to 5 %).  An index that is
// the sum of two with disjoint bits has the sum of their positions, so the per-element part of a pass folds into
// instruction offsets.
__device__ __forceinline__ constexpr int pad(int idx) { return idx + ((idx >> 5) << 1); }
__device__ __forceinline__ double2 &pair_at(double *lds, int pos) { return *reinterpret_cast<double2 *>(lds + pos); }
template <int LOGN> constexpr int lds_doubles() { return (1 << LOGN) + (1 << (LOGN - 4)); }
// position `pos` of row w of rows that lie one after the other.  A row is more than the 64 KB that an instruction's offset reaches:
// left to itself the compiler adds the distance for every element.
template <int LOGN> __device__ __forceinline__ int row_pos(int w, int pos)
{
    if (w) {
        pos += w * lds_doubles<LOGN>();
        asm("" : "+v"(pos));
    }
    return pos;
}

// element `idx` of a row: a uniform base and a 32-bit byte offset per lane (one register instead of two,
// no 64-bit address arithmetic)
template <class T> __device__ __forceinline__ T at32(const T *base, int idx)
{
    return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + (uint32_t)idx * (uint32_t)sizeof(T));
}

typedef double cg_double2v __attribute__((ext_vector_type(2)));
typedef uint64_t cg_ulong2v __attribute__((ext_vector_type(2)));
template <class T> __device__ __forceinline__ void put32(T *base, int idx, T v)
{
    *reinterpret_cast<T *>(reinterpret_cast<char *>(base) + (uint32_t)idx * (uint32_t)sizeof(T)) = v;
}
// Element tid of a row at a uniform address, in the form of a load that takes both: left to itself the compiler
// adds the lane's offset first and carries one 64-bit vector address per row.
template <class T> __device__ __forceinline__ T at_lane(const T *base, int tid)
{
    auto g = (const T __attribute__((address_space(1))) *)base;
    uint32_t off = (uint32_t)tid * (uint32_t)sizeof(T);
    asm("" : "+s"(g));
    asm("" : "+v"(off));
    return *(const T __attribute__((address_space(1))) *)((const char __attribute__((address_space(1))) *)g + off);
}
template <class T> __device__ __forceinline__ void put_lane(T *base, int tid, T v)
{
    auto g = (T __attribute__((address_space(1))) *)base;
    uint32_t off = (uint32_t)tid * (uint32_t)sizeof(T);
    asm("" : "+s"(g));
    asm("" : "+v"(off));
    *(T __attribute__((address_space(1))) *)((char __attribute__((address_space(1))) *)g + off) = v;
}
// a uniform value, kept in scalar registers from here on
__device__ __forceinline__ double pinned(double x)
{
    asm volatile("" : "+s"(x));
    return x;
}
// Constants that are read where they are used: kept for a whole kernel with several transforms they do not
// fit the scalar registers.
template <class T> __device__ __forceinline__ const T *opaque_const(const T *p)
{
    auto g = (const T __attribute__((address_space(4))) *)p;
    asm volatile("" : "+s"(g));
    return (const T *)g;
}

// root: the sub-transform at node `root` of the forward transform's tree (1: a whole row)
template <int LOGN, int E, int PASS, bool HI_ZERO>
__device__ __forceinline__ void load_tw(const double *__restrict__ tw, int tid, double *twr, int root = 1)
{
    using P = Plan<LOGN, E>;
    constexpr int R = P::R[PASS];
    constexpr int S0 = stage_start<LOGN, E, PASS>();
    constexpr int L = LOGN - S0 - R;
    constexpr int G = E >> R;
    constexpr int PER = (1 << R) - 1;
    static_assert(G * PER <= TWREGS, "twiddle register file too small");
#pragma unroll
    for (int g = 0; g < G; g++) {
        int hi = HI_ZERO ? 0 : (group_index<LOGN, E, PASS>(tid, g) >> L);
        // with L >= 6 all 64 lanes of a wave share hi: say so, and the factors come in through
        // the scalar cache instead of one vector load per lane
        if (!HI_ZERO && PASS > 0 && L >= 6) hi = __builtin_amdgcn_readfirstlane(hi);
#pragma unroll
        for (int u = 0; u < R; u++)
#pragma unroll
            for (int j = 0; j < (1 << u); j++)
                twr[g * PER + (1 << u) - 1 + j] = at32(tw + (root << (S0 + u)) + j, hi << u);
    }
}

// ---------------------------------------------------------------------------
// Workgroups are handed to the 8 XCDs round-robin (physical index p runs on XCD p % 8), each
// with its own L2.  Rows that read the same operand are neighbours in logical order, in groups
// of S (the loader's share()); this bijection on [0, nwg) gives every XCD whole groups, so the
// operand comes from HBM once and from that XCD's L2 afterwards: within each full block of 8*S
// physical indices, XCD x takes the logical rows block*8S + x*S ... + S-1.  (Grids are multiples
// of 8 whenever a workgroup walks over more than one row.)
// ---------------------------------------------------------------------------
__device__ __forceinline__ int xcd_row(int p, int nwg, int S)
{
    const int blk = 8 * S;
    const int full = nwg - nwg % blk;
    if (S == 1 || p >= full) return p;
    const int b = p / blk, w = p - b * blk;
    return b * blk + (w & 7) * S + (w >> 3);
}

// ---------------------------------------------------------------------------
// The transform kernels are persistent: a workgroup walks over rows
// wg = blockIdx.x, blockIdx.x + gridDim.x, ... and, while it transforms one row,
// the raw words of its next row are already on their way into registers.
//
// Loader interface (LD):
//   kRaw                       64-bit words fetched per element
//   kPrefetch                  fetch the next row during the current one (else fetch in slices at use)
//   kScatter                   forward only: elements are placed into LDS at place(idx) before pass 0
//   prime(wg, C)               prime index of row wg
//   dst_limb(wg, C)            forward only: destination row
//   fetch(wg, idx, C, raw)     issue the loads of element idx (no arithmetic on the loaded words)
//   finish(raw, wg, idx, m, C) element value, |x| <= FWD_IN 2^50 (forward) or < 2^53 (inverse)
//
// Element ownership: CHUNKED = false: element it of a thread is tid + it * T
// (pass 0); CHUNKED = true: (wave << chunk_log) + lane + 64 * it (the wave's chunk).
// Both put consecutive lanes on consecutive addresses.
// ---------------------------------------------------------------------------
// element `it` of a thread in the chunked ownership: a lane takes pairs of neighbouring elements of
// its wave's chunk, so that every operand comes in (and every result goes out) 16 bytes per lane.
template <int E> __device__ __forceinline__ int chunk_elem(int tid, int it)
{
    return ((tid >> 6) << chunk_log<E>()) + 2 * (tid & 63) + (it & 1) + 128 * (it >> 1);
}

template <int LOGN, int E, bool CHUNKED, class LD>
__device__ __forceinline__ void fetch_row(const LD &ld, int wg, int tid, const DevConst *C,
                                          uint64_t (&raw)[E][LD::kRaw])
{
    constexpr int T = (1 << LOGN) / E;
#pragma unroll
    for (int it = 0; it < E; it++) ld.fetch(wg, CHUNKED ? chunk_elem<E>(tid, it) : tid + it * T, C, raw[it]);
}

// Loaders whose element is a sum over several rounds of fetches (ld.rounds() of them, each with
// ld.fetch_round / ld.finish, the partial sums joined by ld.join) are marked here.
template <class LD> struct ld_rounds { static constexpr bool value = false; };

// Loaders that lift kRaw residue rows to one (row ld.source(target, q) counted from ld.row is word q) are marked
// here: row addresses and the target are worked out once per row.
template <class LD> struct ld_lifts { static constexpr bool value = false; };

// Loaders of half rows are marked here: prime() is 2 r + h, half h of prime r.
template <class LD> struct ld_half { static constexpr bool value = false; };
// Loaders of products' operands: those of N = 16384 are half rows.
template <class LD> struct ld_no_16384 { static constexpr bool value = false; };
// Loaders whose launches always have more rows than compute units.
template <class LD> struct fwd_many { static constexpr bool value = false; };
// Transforms on their own (callers' rows in, rows out), which may use priorities (fwd_pass).
template <class LD, class ST> struct row_alone { static constexpr bool value = false; };

// Loaders that do not prefetch fetch and finish a row in slices, so that at most about 32 raw
// words are live per thread however many words an element needs.
template <int LOGN, int E, bool CHUNKED, class LD, class F>
__device__ __forceinline__ void load_row_now(const LD &ld, int wg, int tid, const ModD m, const DevConst *C, F &&sink)
{
    constexpr int T = (1 << LOGN) / E;
    constexpr int CH0 = LD::kRaw <= 2 ? (ld_rounds<LD>::value ? 8 : 16)
                                      : (LD::kRaw <= 4 ? (E >= 16 && CHUNKED ? 4 : 8) : (E >= 16 && CHUNKED ? 2 : 4));
    constexpr int CH = CH0 < E ? CH0 : E;
    auto at = [&](int it) { return CHUNKED ? chunk_elem<E>(tid, it) : tid + it * T; };
    if constexpr (ld_rounds<LD>::value) {
        const int nr = ld.rounds();
#pragma unroll
        for (int c0 = 0; c0 < E; c0 += CH) {
            double sum[CH];
#pragma unroll
            for (int i = 0; i < CH; i++) sum[i] = 0.0;
            for (int r = 0; r < nr; r++) {
                uint64_t rw[CH][LD::kRaw];
#pragma unroll
                for (int i = 0; i < CH; i++) ld.fetch_round(wg, at(c0 + i), r, C, rw[i]);
#pragma unroll
                for (int i = 0; i < CH; i++) sum[i] = ld.join(sum[i], ld.finish(rw[i], wg, at(c0 + i), m, C), m);
            }
#pragma unroll
            for (int i = 0; i < CH; i++) sink(c0 + i, at(c0 + i), sum[i]);
            __builtin_amdgcn_sched_barrier(0);
        }
        return;
    }
    if constexpr (ld_lifts<LD>::value) {
        static_assert(!CHUNKED, "pass-0 ownership");
        const uint64_t *row = ld.row(wg, C);
        const int j = ld.target(wg, C);
#pragma unroll
        for (int c0 = 0; c0 < E; c0 += CH) {
            uint64_t rw[CH][LD::kRaw];
#pragma unroll
            for (int i = 0; i < CH; i++)
#pragma unroll
                for (int q = 0; q < LD::kRaw; q++)
                    rw[i][q] = at_lane(row + ((size_t)ld.source(j, q) << LOGN) + (c0 + i) * T, tid);
            // the constants are read anew for every slice: kept from slice to slice they do not fit the
            // scalar registers and push the row out of the vector registers
            const DevConst *Cs = opaque_const(C);
#pragma unroll
            for (int i = 0; i < CH; i++) sink(c0 + i, tid + (c0 + i) * T, ld.lift(rw[i], j, m, Cs));
            __builtin_amdgcn_sched_barrier(0);
        }
        return;
    }
#pragma unroll
    for (int c0 = 0; c0 < E; c0 += CH) {
        uint64_t rw[CH][LD::kRaw];
#pragma unroll
        for (int i = 0; i < CH; i++) ld.fetch(wg, at(c0 + i), C, rw[i]);
#pragma unroll
        for (int i = 0; i < CH; i++) sink(c0 + i, at(c0 + i), ld.finish(rw[i], wg, at(c0 + i), m, C));
        // keep the slices apart: hoisting the next slice's loads above this one's arithmetic
        // would bring back the register pressure the slicing is there to avoid
        __builtin_amdgcn_sched_barrier(0);
    }
}

// ---------------------------------------------------------------------------
// forward transform
// ---------------------------------------------------------------------------
// storers that keep the row in LDS (told the element's number in chunk_elem order, not a row)
template <class ST> struct st_in_place { static constexpr bool value = false; };
// the storer of a transform whose results stay in registers, in chunk_elem order
struct StRegs {
    double *out;
    __device__ __forceinline__ void store(int it, int, double v, const ModD) const { out[it] = v; }
};
template <> struct st_in_place<StRegs> { static constexpr bool value = true; };
template <class ST> struct st_regs { static constexpr bool value = false; };
template <> struct st_regs<StRegs> { static constexpr bool value = true; };
// results of a half row of an inverse transform, whose last stage is still to come
struct StHalfRegs : StRegs {};
template <> struct st_regs<StHalfRegs> { static constexpr bool value = true; };

// prio: a wave's priority falls from pass to pass between two barriers, so that those behind catch up and all reach the
// barrier about together.  (Equal priorities let the oldest wave issue first: it runs ahead and then waits.)  Worth 2 to 7 %
// where nothing but such rows is on the chip, so callers' transforms (row_alone), plaintext products and appends, sums of
// products and half rows have it.  Beside other kernels, whose priority is 0, it can hold these up: with priorities in every transform
// a step of twelve heads went from 422 to 430 us, with those of the sums at N = 4096 one of sixteen from 175 to 190, and neither has
// it.  The appends, the sums at N = 8192 and the half rows run beside a step's other branches too, where it is neither gain
// nor loss: steps of 4 to 16 heads at all three N, with each of them on and off, differ by less than 1 % either way, as two runs of
// one library do (12 x 4 in rounds 449 / 449 us, chains 674 / 674; 16 x 3 at N = 16384 1890 / 1902, chains 3219 / 3234).
// U: rows of one prime taken through the pass together, row u in in[u E ...] or u * lds_doubles() further on in LDS.  They share the
// pass's factors and its barrier.
template <int LOGN, int E, int PASS, bool FROM_REGS, int U = 1, int IN = (int)(100 * FWD_IN), class ST>
__device__ __forceinline__ void fwd_pass(double *lds, const double *in, const ST &st, int tid,
                                         const double *__restrict__ tw, const double *twr, double *twr_next,
                                         const ModD m, int dst_limb, bool prio = false, int root = 1)
{
    using P = Plan<LOGN, E>;
    constexpr int R = P::R[PASS];
    constexpr int S0 = stage_start<LOGN, E, PASS>();
    constexpr int L = LOGN - S0 - R;          // index bits below this pass's R bits
    constexpr int G = E >> R;                 // independent radix-2^R groups per thread
    constexpr int PER = (1 << R) - 1;
    constexpr bool first = PASS == 0, last = PASS == P::NP - 1;
    constexpr bool cross = PASS < P::NC;      // pairs elements owned by different waves
    constexpr bool do_red = FwdBound<LOGN, E, PASS, IN>::reduce;
    static_assert(FwdBound<LOGN, E, PASS, IN>::out < 8.0, "lazy bound exceeds 2^53");
    static_assert(!FROM_REGS || (first && L + R == LOGN), "register input only for the first pass");
    static_assert(cross || L + R <= chunk_log<E>(), "wave-local passes must stay inside one chunk");
    static_assert(!last || !cross, "the last pass must be wave-local (chunk-wise copy-out)");
    static_assert(U == 1 || st_regs<ST>::value, "rows together stay in registers");
    constexpr int ROW = lds_doubles<LOGN>();
    if (prio) __builtin_amdgcn_s_setprio(PASS <= 1 ? 3 : last ? 1 : 2);
    double v[U][G][1 << R];
    int base[G];
#pragma unroll
    for (int g = 0; g < G; g++) {
        const int gidx = group_index<LOGN, E, PASS>(tid, g);
        const int lo = gidx & ((1 << L) - 1);
        const int hi = first ? 0 : (gidx >> L);
        base[g] = (hi << (L + R)) | lo;
    }
#pragma unroll
    for (int w = 0; w < U; w++)
#pragma unroll
        for (int g = 0; g < G; g++) {
            const int pb = row_pos<LOGN>(w, pad(base[g]));
#pragma unroll
            for (int c = 0; c < (1 << R); c++) {
                // first pass: element base + (c << L) = tid + (g + c*G) * T is fetched element g + c*G
                if (FROM_REGS) v[w][g][c] = in[w * E + g + c * G];
                else if (L > 0) v[w][g][c] = lds[pb + pad(c << L)];
                else if (c % 2 == 0) {
                    const double2 x = pair_at(lds, pb + c);
                    v[w][g][c] = x.x;
                    v[w][g][c + 1] = x.y;
                }
            }
        }
#pragma unroll
    for (int w = 0; w < U; w++)
#pragma unroll
        for (int g = 0; g < G; g++) {
            if (do_red) {
#pragma unroll
                for (int c = 0; c < (1 << R) / 2; c++) v[w][g][c] = red(v[w][g][c], m);
            }
#pragma unroll
            for (int u = 0; u < R; u++) {
                const int half = 1 << (R - 1 - u);
#pragma unroll
                for (int c = 0; c < (1 << R); c++) {
                    if (c & half) continue;
                    bfly_fwd(v[w][g][c], v[w][g][c + half], twr[g * PER + (1 << u) - 1 + (c >> (R - u))], m);
                }
            }
        }
    // a last pass on pairs of neighbours leaves them where chunk_elem order has them: no trip to LDS
    if constexpr (last && R == 1 && st_regs<ST>::value) {
#pragma unroll
        for (int w = 0; w < U; w++)
#pragma unroll
            for (int g = 0; g < G; g++) {
                st.store(w * E + 2 * g, 0, v[w][g][0], m);
                st.store(w * E + 2 * g + 1, 0, v[w][g][1], m);
            }
        return;
    }
    // fetch the next pass's factors while this pass's results drain to LDS
    if constexpr (U > 1) __builtin_amdgcn_sched_barrier(0);     // (sooner they take registers that two rows need)
    if constexpr (!last) load_tw<LOGN, E, PASS + 1, false>(tw, tid, twr_next, root);
#pragma unroll
    for (int w = 0; w < U; w++)
#pragma unroll
        for (int g = 0; g < G; g++) {
            const int pb = row_pos<LOGN>(w, pad(base[g]));
#pragma unroll
            for (int c = 0; c < (1 << R); c++) {
                if (L > 0) lds[pb + pad(c << L)] = v[w][g][c];
                else if (c % 2 == 0) pair_at(lds, pb + c) = make_double2(v[w][g][c], v[w][g][c + 1]);
            }
        }
    if constexpr (cross) lds_barrier();
    else wave_sync();
    if constexpr (last) {
        // results leave through LDS so that consecutive lanes write consecutive addresses; each
        // wave copies out its own chunk
        // (a lane takes pairs of neighbouring elements: 16 bytes per lane and store)
#pragma unroll
        for (int it = 0; it < U * E; it += 2) {
            const int idx = chunk_elem<E>(tid, it % E);
            const double2 w = pair_at(lds, it / E * ROW + pad(idx));
            if constexpr (st_in_place<ST>::value) {
                st.store(it, idx, w.x, m);
                st.store(it + 1, idx + 1, w.y, m);
            } else {
                st.store(dst_limb, idx, w.x, m);
                st.store(dst_limb, idx + 1, w.y, m);
            }
        }
    }
}

template <int LOGN, int E, class LD, class ST>
__global__ void __launch_bounds__((1 << LOGN) / E, (min_waves<LOGN, E>()))
ntt_fwd_kernel(LD ld, ST st, const double *__restrict__ tw_all, const DevConst *__restrict__ C, int nwg)
{
    __shared__ __align__(16) double lds[lds_doubles<LOGN>()];
    constexpr bool PF = LD::kPrefetch && prefetch_rows<LOGN, E>();
    constexpr int T = (1 << LOGN) / E;
    constexpr int NP = Plan<LOGN, E>::NP;
    // Rows for a round and a half of workgroups (us, N = 8192: 1000 rows 32.0 -> 31.1, 4000: 132 -> 123, 16384: 488 -> 471;
    // 1500 rows of 4096: 22.8 -> 21.5; 1000 of 16384: 66.2 -> 63.3).  Below, a gain and a loss by turns, as what is left
    // over runs on nearly idle units: 60 rows of 8192 7.9 -> 7.5, 250: 8.9 -> 9.3, 512: 17.3 -> 17.0, 600: 21.3 -> 22.5.
    const bool prio = row_alone<LD, ST>::value && 2 * nwg >= 3 * (int)gridDim.x;
    const int tid = threadIdx.x;
    const int S = ld.share(C);
    int p = blockIdx.x;
    int wg = xcd_row(p, nwg, S);
    // loaders that scatter into LDS before pass 0 are free in which elements a thread brings in:
    // they use the chunked ownership; the others bring in what pass 0 works on in registers
    constexpr bool CH = LD::kScatter;
    uint64_t raw[PF ? E : 1][LD::kRaw];
    if constexpr (PF) fetch_row<LOGN, E, CH>(ld, wg, tid, C, raw);
    for (;;) {
        const int pr = ld.prime(wg, C);
        const ModD m = C->mod[ld_half<LD>::value ? pr >> 1 : pr];
        const double *tw = tw_all + ((size_t)pr << LOGN);
        const int dl = ld.dst_limb(wg, C);
        double twa[TWREGS], twb[TWREGS];
        if constexpr (PF) load_tw<LOGN, E, 0, true>(tw, tid, twa);
        double in[E];
        p += (int)gridDim.x;
        const bool more = p < nwg;
        const int wg_next = more ? xcd_row(p, nwg, S) : 0;
        if constexpr (PF) {
#pragma unroll
            for (int it = 0; it < E; it++)
                in[it] = ld.finish(raw[it], wg, CH ? chunk_elem<E>(tid, it) : tid + it * T, m, C);
            if (more) fetch_row<LOGN, E, CH>(ld, wg_next, tid, C, raw);
        } else {
            load_row_now<LOGN, E, CH>(ld, wg, tid, m, C, [&](int it, int, double v) { in[it] = v; });
            load_tw<LOGN, E, 0, true>(tw, tid, twa);     // (scalar registers that the loader's constants need)
        }
        if constexpr (LD::kScatter) {
#pragma unroll
            for (int it = 0; it < E; it++) lds[pad(ld.place(chunk_elem<E>(tid, it), 1 << LOGN))] = in[it];
            lds_barrier();
            fwd_pass<LOGN, E, 0, false>(lds, in, st, tid, tw, twa, twb, m, dl, prio);
        } else {
            fwd_pass<LOGN, E, 0, true>(lds, in, st, tid, tw, twa, twb, m, dl, prio);
        }
        fwd_pass<LOGN, E, 1, false>(lds, in, st, tid, tw, twb, twa, m, dl, prio);
        fwd_pass<LOGN, E, 2, false>(lds, in, st, tid, tw, twa, twb, m, dl, prio);
        if constexpr (NP > 3) fwd_pass<LOGN, E, 3, false>(lds, in, st, tid, tw, twb, twa, m, dl, prio);
        if constexpr (NP > 4) fwd_pass<LOGN, E, 4, false>(lds, in, st, tid, tw, twa, twb, m, dl, prio);
        if (!more) break;
        wg = wg_next;
        lds_barrier();   // the copy-out reads of this row precede the next row's LDS writes
    }
}

// ---------------------------------------------------------------------------
// inverse transform (passes in reverse order; N^-1 folded into the last stage)
// ---------------------------------------------------------------------------
// storers that add to what the destination holds (fetch() brings it in)
template <class ST> struct st_adds { static constexpr bool value = false; };
template <class ST> struct st_adds<const ST> : st_adds<ST> {};
template <class ST> struct st_adds<const ST &> : st_adds<ST> {};
// storers of rows without the factor N^-1 (scale_kernel has it among its constants): bound of the results, in hundredths
template <class ST> struct st_unscaled { static constexpr int value = 0; };
template <class ST> struct st_unscaled<const ST> : st_unscaled<ST> {};
template <> struct st_unscaled<StHalfRegs> { static constexpr int value = 365; };
// Loaders of inverse transforms: bound of what they deliver (InvBound's IN).  With it the first pass reduces what its plan asks for, and a
// factor of a product need not be reduced to keep the other bounds: with N^-1 left to the scaling a product's workgroup (mul_row_kernel,
// three primes) has 5110 FP64 instructions a thread -> 4978, one of a sum 4162 -> 4066, a plaintext product 1066 -> 1046.
// 768 products and relinearisations at N = 8192 1830 -> 1780 us, 128 appends of 24 caches (with the stores' addresses in scalar
// registers and one reduction for sum and result) 1928 -> 1882.
template <class LD> struct ld_in { static constexpr int value = 0; };

// from != null: the first pass takes its elements from registers, in chunk_elem order
// early: the first eight words that a storer adds to
// U: rows of one prime together, as in fwd_pass; results of row u leave as row wg + u * row_step, or to out[u E ...]
template <int LOGN, int E, int PASS, int IN = 0, int U = 1, class ST>
__device__ __forceinline__ void inv_pass(double *lds, const ST &st, int wg, int tid,
                                         const double *__restrict__ itw, const double *twr, double *twr_next,
                                         const ModD m, int pr, const DevConst *C, const double *from = nullptr,
                                         const uint64_t *early = nullptr, bool prio = false, int row_step = 0,
                                         int root = 1)
{
    using P = Plan<LOGN, E>;
    constexpr int R = P::R[PASS];
    constexpr int S0 = stage_start<LOGN, E, PASS>();
    constexpr int L = LOGN - S0 - R;
    constexpr int G = E >> R;
    constexpr int PER = (1 << R) - 1;
    constexpr bool last = PASS == 0;
    constexpr bool cross = PASS < P::NC;
    constexpr int unscaled = st_unscaled<ST>::value;
    constexpr InvPlan<R> plan = inv_plan<R>(InvBound<LOGN, E, PASS, IN>::in, !last ? 0 : unscaled ? 2 : 1, 0.01 * unscaled);
    static_assert(plan.out <= LAZY_MAX, "lazy bound exceeds 2^53");
    static_assert(cross || L + R <= chunk_log<E>(), "wave-local passes must stay inside one chunk");
    if (prio) __builtin_amdgcn_s_setprio(PASS < 2 ? 3 : PASS == P::NP - 1 ? 2 : PASS == P::NP - 2 ? 1 : 0);
    double v[U][G][1 << R];
    int base[G];
#pragma unroll
    for (int g = 0; g < G; g++) {
        // the last pass stores straight to global memory and all its groups share their twiddles:
        // with an even number of groups a thread takes neighbouring ones (16 bytes per lane and store)
        const int gidx = (last && G % 2 == 0) ? 2 * tid + (g & 1) + 2 * ((1 << LOGN) / E) * (g >> 1)
                                              : group_index<LOGN, E, PASS>(tid, g);
        const int lo = gidx & ((1 << L) - 1);
        const int hi = last ? 0 : (gidx >> L);
        base[g] = (hi << (L + R)) | lo;
    }
#pragma unroll
    for (int w = 0; w < U; w++)
#pragma unroll
        for (int g = 0; g < G; g++) {
            const int pb = row_pos<LOGN>(w, pad(base[g]));
#pragma unroll
            for (int c = 0; c < (1 << R); c++) {
                if (R == 1 && from) v[w][g][c] = from[w * E + 2 * g + c];
                else if (L > 0) v[w][g][c] = lds[pb + pad(c << L)];
                else if (c % 2 == 0) {
                    const double2 x = pair_at(lds, pb + c);
                    v[w][g][c] = x.x;
                    v[w][g][c + 1] = x.y;
                }
            }
        }
    static_assert(!(last && st_regs<ST>::value) || G == 1, "one group per thread in the last pass");
    constexpr bool adds = last && st_adds<ST>::value;
    static_assert(!adds || (U == 1 && G == 1 && (1 << R) % 8 == 0), "eight elements of the one group at a time");
    uint64_t old[adds ? 8 : 1];
#pragma unroll
    for (int w = 0; w < U; w++)
#pragma unroll
        for (int g = 0; g < G; g++) {
            double (&x)[1 << R] = v[w][g];
            if (PASS == P::NP - 1 && !IN) {
#pragma unroll
                for (int c = 0; c < (1 << R); c++) x[c] = red(x[c], m);
            }
#pragma unroll
            for (int u = R - 1; u >= 0; u--) {
                const int half = 1 << (R - 1 - u);
#pragma unroll
                for (int c = 0; c < (1 << R); c++)
                    if (plan.before[R - 1 - u][c]) x[c] = red(x[c], m);
#pragma unroll
                for (int c = 0; c < (1 << R); c++) {
                    if (c & half) continue;
                    if (last && u == 0 && !unscaled) {
                        // stage 0: single twiddle; fold N^-1 into both outputs
                        const double d = x[c] - x[c + half];
                        x[c] = mulmod(x[c] + x[c + half], C->ninv[pr], m);
                        x[c + half] = mulmod(d, C->itw1_ninv[pr], m);
                    } else {
                        bfly_inv(x[c], x[c + half], twr[g * PER + (1 << u) - 1 + (c >> (R - u))], m);
                    }
                }
            }
#pragma unroll
            for (int c = 0; c < (1 << R); c++)
                if (plan.after[c]) x[c] = red(x[c], m);
        }
    if constexpr (!last) {
        if constexpr (PASS == 1) load_tw<LOGN, E, 0, true>(itw, tid, twr_next, root);
        else load_tw<LOGN, E, PASS - 1, false>(itw, tid, twr_next, root);
    }
#pragma unroll
    for (int w = 0; w < U; w++)
#pragma unroll
        for (int g = 0; g < G; g++) {
            const int pb = row_pos<LOGN>(w, pad(base[g]));
#pragma unroll
            for (int c = 0; c < (1 << R); c++) {
                // the last pass pairs elements N/2 apart with consecutive lanes on consecutive
                // addresses: it stores straight to global memory
                if constexpr (adds) {
                    if (c == 0) {
#pragma unroll
                        for (int i = 0; i < 8; i++) old[i] = early[i];
                    } else if (c % 8 == 0) {
                        st.template fetch<(1 << LOGN) / E>(old, tid, c);
                    }
                }
                if (!last) {
                    if (L > 0) lds[pb + pad(c << L)] = v[w][g][c];
                    else if (c % 2 == 0) pair_at(lds, pb + c) = make_double2(v[w][g][c], v[w][g][c + 1]);
                } else if constexpr (st_adds<ST>::value) st.store(c << L, base[g], v[w][g][c], old[c % 8], m);
                else if constexpr (st_regs<ST>::value) st.store(w * E + c, 0, v[w][g][c], m);     // (element tid + c * T)
                else if constexpr (G == 1) st.store_lane(wg + w * row_step, c << L, base[g], v[w][g][c], m);
                else st.store(wg + w * row_step, base[g] + (c << L), v[w][g][c], m);
            }
        }
    if constexpr (!last) {
        if constexpr (PASS - 1 < P::NC) lds_barrier();   // the next pass reads other waves' elements
        else wave_sync();
    }
}

// rows p, p + step, ... of nwg
template <int LOGN, int E, class LD, class ST>
__device__ __forceinline__ void inv_rows(double *lds, int p, int step, const LD &ld, const ST &st, const double *__restrict__ itw_all,
                                         const DevConst *__restrict__ C, int nwg)
{
    constexpr bool PF = LD::kPrefetch && prefetch_rows<LOGN, E>();
    constexpr int NP = Plan<LOGN, E>::NP, IN = ld_in<LD>::value;
    static_assert(NP - 1 >= Plan<LOGN, E>::NC, "the first inverse pass must be wave-local");
    // (N = 4096, 1500 rows: 24.9 -> 23.6 us, 4096: 57 -> 55.  N = 8192, 512 threads: inv_wide; 1024 threads: 1000 rows 35.7 -> 37.0, 4000 the
    // same; 4000 of 16384: 274 -> 286.)
    const bool prio = (LOGN <= 12 || (LOGN == 13 && E == 16)) && row_alone<LD, ST>::value && 2 * nwg >= 3 * step;
    const int tid = threadIdx.x;
    const int S = ld.share(C);
    int wg = xcd_row(p, nwg, S);
    uint64_t raw[PF ? E : 1][LD::kRaw];
    if constexpr (PF) fetch_row<LOGN, E, true>(ld, wg, tid, C, raw);
    for (;;) {
        const int pr = ld.prime(wg, C);
        const ModD m = C->mod[pr];
        const double *itw = itw_all + ((size_t)pr << LOGN);
        double twa[TWREGS], twb[TWREGS];
        load_tw<LOGN, E, NP - 1, false>(itw, tid, twa);
        {
            // each wave brings in its own chunk (consecutive lanes on consecutive addresses) and
            // re-reads it from LDS in the stride-1 pattern of the first pass
            if constexpr (PF) {
#pragma unroll
                for (int it = 0; it < E; it += 2) {
                    const int idx = chunk_elem<E>(tid, it);
                    pair_at(lds, pad(idx)) =
                        make_double2(ld.finish(raw[it], wg, idx, m, C), ld.finish(raw[it + 1], wg, idx + 1, m, C));
                }
            } else {
                double first = 0.0;     // (elements come in pairs)
                load_row_now<LOGN, E, true>(ld, wg, tid, m, C, [&](int it, int idx, double v) {
                    if (it % 2 == 0) first = v;
                    else pair_at(lds, pad(idx - 1)) = make_double2(first, v);
                });
            }
        }
        p += step;
        const bool more = p < nwg;
        const int wg_next = more ? xcd_row(p, nwg, S) : 0;
        const int orow = ld.out_row(wg, C);
        if constexpr (PF) {
            if (more) fetch_row<LOGN, E, true>(ld, wg_next, tid, C, raw);
        }
        wave_sync();
        // passes NP-1 ... 0; the twiddle buffers alternate
        if constexpr (NP == 5) {
            inv_pass<LOGN, E, 4, IN>(lds, st, orow, tid, itw, twa, twb, m, pr, C, nullptr, nullptr, prio);
            inv_pass<LOGN, E, 3, IN>(lds, st, orow, tid, itw, twb, twa, m, pr, C, nullptr, nullptr, prio);
            inv_pass<LOGN, E, 2, IN>(lds, st, orow, tid, itw, twa, twb, m, pr, C, nullptr, nullptr, prio);
            inv_pass<LOGN, E, 1, IN>(lds, st, orow, tid, itw, twb, twa, m, pr, C, nullptr, nullptr, prio);
            inv_pass<LOGN, E, 0, IN>(lds, st, orow, tid, itw, twa, twb, m, pr, C, nullptr, nullptr, prio);
        } else if constexpr (NP == 4) {
            inv_pass<LOGN, E, 3, IN>(lds, st, orow, tid, itw, twa, twb, m, pr, C, nullptr, nullptr, prio);
            inv_pass<LOGN, E, 2, IN>(lds, st, orow, tid, itw, twb, twa, m, pr, C, nullptr, nullptr, prio);
            inv_pass<LOGN, E, 1, IN>(lds, st, orow, tid, itw, twa, twb, m, pr, C, nullptr, nullptr, prio);
            inv_pass<LOGN, E, 0, IN>(lds, st, orow, tid, itw, twb, twa, m, pr, C, nullptr, nullptr, prio);
        } else {
            inv_pass<LOGN, E, 2, IN>(lds, st, orow, tid, itw, twa, twb, m, pr, C, nullptr, nullptr, prio);
            inv_pass<LOGN, E, 1, IN>(lds, st, orow, tid, itw, twb, twa, m, pr, C, nullptr, nullptr, prio);
            inv_pass<LOGN, E, 0, IN>(lds, st, orow, tid, itw, twa, twb, m, pr, C, nullptr, nullptr, prio);
        }
        if (!more) break;
        wg = wg_next;
        lds_barrier();   // pass 0's LDS reads precede the next row's LDS writes
    }
}
template <int LOGN, int E, class LD, class ST>
__global__ void __launch_bounds__((1 << LOGN) / E, (min_waves<LOGN, E>()))
ntt_inv_kernel(LD ld, ST st, const double *__restrict__ itw_all, const DevConst *__restrict__ C, int nwg)
{
    __shared__ __align__(16) double lds[lds_doubles<LOGN>()];
    inv_rows<LOGN, E>(lds, (int)blockIdx.x, (int)gridDim.x, ld, st, itw_all, C, nwg);
}

// Inverse loaders marked here run with 16 elements per thread at N = 8192 where there are more rows than this many halves of the compute units,
// like the forward transforms (two co-resident 512-thread workgroups per compute unit).  It pays for the tensor
// product, whose launches are large then, and for callers' rows (us, 1024 threads / 512: 400 rows 16.9 / 15.6, 512: 18.8 / 17.8, 700: 25.9 / 23.8,
// 1000: 35.5 / 33.0, 2000: 72 / 65, 4323: 155 / 136, 16384: 565 / 488, without priorities 522); the key-switch inner product is
// launched over a few hundred rows at a time and finishes a row sooner on 1024 threads.
template <class LD> struct inv_wide { static constexpr int value = 0; };

// ---------------------------------------------------------------------------
// exact base conversion helpers (per coefficient, registers only)
// ---------------------------------------------------------------------------
// The size of the source basis is a template argument everywhere: with a run-time size every step of
// these loops is a branch and the scaled configuration's mod-down (two special primes) took four times
// as long.
//
// ms: the source basis' moduli (consecutive ones of the context's).  x[0..NS) canonical residues -> mixed-radix digits 0 <= a_i < s_i of the integer in [0, S)
template <int NS>
__device__ __forceinline__ void garner(const ConvTab &T, const ModD *ms, const double (&x)[NS], double (&a)[NS])
{
    a[0] = x[0];
#pragma unroll
    for (int j = 1; j < NS; j++) {
        const ModD mj = ms[j];
        double v = x[j];
#pragma unroll
        for (int i = 0; i < j; i++) v = mulmod(v - a[i], T.inv[i][j], mj);
        a[j] = canon(v, mj);
    }
}
// x[0..NS) residues, |x_j| <= 2p -> digits |a_i| <= (s_i - 1)/2.  These balanced digits represent exactly
// the integers of magnitude at most (S - 1)/2: the centred representative, without the comparison with
// S/2 and without making the digits canonical.  red() picks the balanced residue exactly here: its
// quotient x u is off by less than 1.25 * 2^-52 up to |x u| = 2, and the residues next to an odd multiple of p/2 are
// 2^-51 away.
template <int NS, class TAB>
__device__ __forceinline__ void garner_balanced(const TAB &T, const ModD *ms, const double (&x)[NS], double (&a)[NS])
{
    a[0] = red(x[0], ms[0]);
#pragma unroll
    for (int j = 1; j < NS; j++) {
        const ModD mj = ms[j];
        double v = x[j];
#pragma unroll
        for (int i = 0; i < j; i++) v = mulmod(v - a[i], T.inv[i][j], mj);
        a[j] = red(v, mj);
    }
}
// residue of the integer modulo target jt (mt); lazy, |.| < 1.25 * 2^50 with balanced digits, < 2.1 * 2^50 with
// canonical ones
template <int NS, class TAB>
__device__ __forceinline__ double horner(const TAB &T, const ModD mt, const double (&a)[NS], int jt)
{
    double acc = a[NS - 1];
#pragma unroll
    for (int i = NS - 2; i >= 0; i--) acc = mulmod(acc, T.s_mod_t[i][jt], mt) + a[i];
    return acc;
}

// ---------------------------------------------------------------------------
// loaders / storers for the transforms
// ---------------------------------------------------------------------------
struct StF64 {      // forward output: lazy doubles
    double *base;
    __device__ __forceinline__ void store(int limb, int idx, double v, const ModD) const
    {
        base[((size_t)limb << logn) + idx] = v;
    }
    int logn;
};
struct StF64Red {   // forward output reduced to |x| <= p/2 (prepared keys and plaintexts)
    double *base;
    int logn;
    __device__ __forceinline__ void store(int limb, int idx, double v, const ModD m) const
    {
        base[((size_t)limb << logn) + idx] = red(v, m);
    }
};
struct StU64 {      // forward output: canonical uint64 (public transform entry point)
    uint64_t *base;
    int logn;
    __device__ __forceinline__ void store(int limb, int idx, double v, const ModD m) const
    {
        base[((size_t)limb << logn) + idx] = f64_to_u64(canon(v, m));
    }
};

__device__ __forceinline__ uint64_t f64_bits(double x)
{
    union { double d; uint64_t u; } v;
    v.d = x;
    return v.u;
}
__device__ __forceinline__ double bits_f64(uint64_t x)
{
    union { double d; uint64_t u; } v;
    v.u = x;
    return v.d;
}

// rows of uint64 residues, row w uses prime tab[w] (tab != null) or w % pmod
struct LdRowsU64 {
    static constexpr int kRaw = 1;
    static constexpr bool kPrefetch = true;
    static constexpr bool kScatter = false;
    const uint64_t *src;
    const uint32_t *tab;
    int pmod, logn;
    __device__ __forceinline__ int prime(int wg, const DevConst *) const { return tab ? (int)tab[wg] : wg % pmod; }
    __device__ __forceinline__ int share(const DevConst *) const { return 1; }
    __device__ __forceinline__ int dst_limb(int wg, const DevConst *) const { return wg; }
    __device__ __forceinline__ void fetch(int wg, int idx, const DevConst *, uint64_t *raw) const
    {
        raw[0] = src[((size_t)wg << logn) + idx];
    }
    __device__ __forceinline__ double finish(const uint64_t *raw, int, int, const ModD, const DevConst *) const
    {
        return u64_to_f64(raw[0]);
    }
};
template <> struct row_alone<LdRowsU64, StU64> { static constexpr bool value = true; };

// the same with the first n_first rows from `first` and the others, counted from there on, from `src`
struct LdRowsFirst {
    static constexpr int kRaw = 1;
    static constexpr bool kPrefetch = true;
    static constexpr bool kScatter = false;
    const uint64_t *first, *src;
    int n_first, pmod, logn;
    __device__ __forceinline__ int prime(int wg, const DevConst *) const { return wg % pmod; }
    __device__ __forceinline__ int share(const DevConst *) const { return 1; }
    __device__ __forceinline__ int dst_limb(int wg, const DevConst *) const { return wg; }
    __device__ __forceinline__ void fetch(int wg, int idx, const DevConst *, uint64_t *raw) const
    {
        raw[0] = (wg < n_first ? first + ((size_t)wg << logn) : src + ((size_t)(wg - n_first) << logn))[idx];
    }
    __device__ __forceinline__ double finish(const uint64_t *raw, int, int, const ModD, const DevConst *) const
    {
        return u64_to_f64(raw[0]);
    }
};

// Inputs of a batch of tensor products.  The source ciphertexts are the n_a "a" operands followed
// by the `batch` "b" operands; polynomial pp = 2 * ciphertext + component.  Every polynomial is
// transformed once over the k ciphertext primes (LdMulQ) and the l auxiliary primes (LdMulAux) into
// ntt[pp][k+l][N]; an a operand shared by several products is transformed once.
struct MulSrc {
    const uint64_t *cta, *ctb;
    int n_a, b_group, b_stride, logn;   // b ciphertext of unit u: (u / b_group) * b_stride + u % b_group
    int dst_strided;                    // transformed rows land at the source's (strided) ciphertext index
    __device__ __forceinline__ int dst_poly(int pp) const
    {
        if (!dst_strided) return pp;
        const int u = (pp >> 1) - n_a;
        return 2 * ((u / b_group) * b_stride + u % b_group) + (pp & 1);
    }
    __device__ __forceinline__ const uint64_t *poly(int pp, int k) const
    {
        // (no branch: loaders ask for the row once per element and leave it to the compiler to do so once)
        const int ct = pp >> 1, comp = pp & 1, u = ct < n_a ? 0 : ct - n_a;
        const int idx = ct < n_a ? ct : (u / b_group) * b_stride + u % b_group;
        return (ct < n_a ? cta : ctb) + (((size_t)(2 * idx + comp) * k) << logn);
    }
};
// operands of mul_row_kernel: x in coefficients, unit u's at x + (u / x_group) * x_stride + u % x_group (in
// ciphertexts); y likewise in coefficients, or transformed rows [ciphertext][2][k+l][N].  Lifted operands: rows of
// doubles, k = 2 (k + l) half rows of 2^logn to a polynomial.
struct MulRowArgs {
    const uint64_t *x, *y;
    const double *yhat;
    int x_group, x_stride, x_div, y_group, y_stride, y_div, k, logn;
    static __device__ __forceinline__ int index(int u, int group, int stride, int div)
    {
        u /= div;
        return u / group * stride + u % group;
    }
    __device__ __forceinline__ const uint64_t *x_poly(int u, int c) const
    {
        return x + ((size_t)(index(u, x_group, x_stride, x_div) * 2 + c) * k << logn);
    }
    __device__ __forceinline__ const uint64_t *y_poly(int u, int c) const
    {
        return y + ((size_t)(index(u, y_group, y_stride, y_div) * 2 + c) * k << logn);
    }
    __device__ __forceinline__ const double *y_hat(int u, int r, int KL) const
    {
        return yhat + ((size_t)(index(u, y_group, y_stride, y_div) * 2 * KL + r) << logn);
    }
};
struct LdMulQ {     // workgroup -> (pp, ciphertext prime i)
    static constexpr int kRaw = 1;
    static constexpr bool kPrefetch = true;
    static constexpr bool kScatter = false;
    MulSrc src;
    __device__ __forceinline__ int prime(int wg, const DevConst *C) const { return wg % C->k; }
    __device__ __forceinline__ int share(const DevConst *) const { return 1; }
    __device__ __forceinline__ int dst_limb(int wg, const DevConst *C) const
    {
        return src.dst_poly(wg / C->k) * C->KL + wg % C->k;
    }
    __device__ __forceinline__ void fetch(int wg, int idx, const DevConst *C, uint64_t *raw) const
    {
        const int k = C->k;
        raw[0] = src.poly(wg / k, k)[((size_t)(wg % k) << src.logn) + idx];
    }
    __device__ __forceinline__ double finish(const uint64_t *raw, int, int, const ModD, const DevConst *) const
    {
        return u64_to_f64(raw[0]);
    }
};
// workgroup -> (pp, auxiliary prime j): the centred integer lift of each coefficient (exact, via
// mixed-radix digits of its K residues) reduced modulo the auxiliary prime
template <int K>
struct LdMulAux {
    static constexpr int kRaw = K;
    static constexpr bool kPrefetch = false;
    static constexpr bool kScatter = false;
    MulSrc src;
    __device__ __forceinline__ int prime(int wg, const DevConst *C) const { return C->k + wg % C->l; }
    __device__ __forceinline__ int share(const DevConst *C) const { return C->l; }
    __device__ __forceinline__ int dst_limb(int wg, const DevConst *C) const
    {
        return src.dst_poly(wg / C->l) * C->KL + C->k + wg % C->l;
    }
    __device__ __forceinline__ const uint64_t *row(int wg, const DevConst *C) const { return src.poly(wg / C->l, K); }
    __device__ __forceinline__ int target(int wg, const DevConst *C) const { return wg % C->l; }
    static __device__ __forceinline__ int source(int, int q) { return q; }
    static __device__ __forceinline__ double lift(const uint64_t *raw, int j, const ModD mb, const DevConst *C)
    {
        double x[K], dg[K];
#pragma unroll
        for (int i = 0; i < K; i++) x[i] = u64_to_f64(raw[i]);
        garner_balanced<K>(C->q2b, C->mod, x, dg);
        return horner<K>(C->q2b, mb, dg, j);
    }
    __device__ __forceinline__ void fetch(int, int, const DevConst *, uint64_t *) const {}
    __device__ __forceinline__ double finish(const uint64_t *, int, int, const ModD, const DevConst *) const { return 0.0; }
};
template <int K> struct ld_lifts<LdMulAux<K>> { static constexpr bool value = true; };
template <> struct ld_no_16384<LdMulQ> { static constexpr bool value = true; };
template <int K> struct ld_no_16384<LdMulAux<K>> { static constexpr bool value = true; };
// (taken with more than two rows of k + l per compute unit, l > k of which are more than one per unit)
template <int K> struct fwd_many<LdMulAux<K>> { static constexpr bool value = true; };

// Both kinds of rows in one launch, for launches that leave compute units free: workgroup -> (pp, prime r of the k + l).
// All K words of a row modulo a ciphertext prime are that row's own: the same line, and the same code.
template <int K>
struct LdMulExt {
    static constexpr int kRaw = K;
    static constexpr bool kPrefetch = false;
    static constexpr bool kScatter = false;
    MulSrc src;
    __device__ __forceinline__ int prime(int wg, const DevConst *) const { return wg % (2 * K + 1); }
    __device__ __forceinline__ int share(const DevConst *) const { return 2 * K + 1; }
    __device__ __forceinline__ int dst_limb(int wg, const DevConst *) const
    {
        return src.dst_poly(wg / (2 * K + 1)) * (2 * K + 1) + wg % (2 * K + 1);
    }
    __device__ __forceinline__ const uint64_t *row(int wg, const DevConst *) const { return src.poly(wg / (2 * K + 1), K); }
    __device__ __forceinline__ int target(int wg, const DevConst *) const { return wg % (2 * K + 1); }
    static __device__ __forceinline__ int source(int r, int q) { return r < K ? r : q; }
    static __device__ __forceinline__ double lift(const uint64_t *raw, int r, const ModD m, const DevConst *C)
    {
        return r < K ? u64_to_f64(raw[0]) : LdMulAux<K>::lift(raw, r - K, m, C);
    }
    __device__ __forceinline__ void fetch(int, int, const DevConst *, uint64_t *) const {}
    __device__ __forceinline__ double finish(const uint64_t *, int, int, const ModD, const DevConst *) const { return 0.0; }
};
template <int K> struct ld_lifts<LdMulExt<K>> { static constexpr bool value = true; };
template <int K> struct ld_no_16384<LdMulExt<K>> { static constexpr bool value = true; };

// half rows that lift_kernel left, transformed in place: workgroup -> (pp, row 2 r + h of 2 (k + l))
struct LdHalf {
    static constexpr int kRaw = 1;
    static constexpr bool kPrefetch = true;
    static constexpr bool kScatter = false;
    const double *rows;
    MulSrc src;
    __device__ __forceinline__ int prime(int wg, const DevConst *C) const { return wg % (2 * C->KL); }
    __device__ __forceinline__ int share(const DevConst *) const { return 1; }
    __device__ __forceinline__ int dst_limb(int wg, const DevConst *C) const
    {
        const int per = 2 * C->KL;
        return src.dst_poly(wg / per) * per + wg % per;
    }
    __device__ __forceinline__ void fetch(int wg, int idx, const DevConst *C, uint64_t *raw) const
    {
        raw[0] = f64_bits(rows[((size_t)dst_limb(wg, C) << (src.logn - 1)) + idx]);
    }
    __device__ __forceinline__ double finish(const uint64_t *raw, int, int, const ModD, const DevConst *) const
    {
        return bits_f64(raw[0]);
    }
};
template <> struct ld_half<LdHalf> { static constexpr bool value = true; };

// key-switch mod-up: workgroup -> (unit b, digit j, target prime r); the digit is
// the integer in [0,Q_j) formed by ALPHA rows of the source ring element, reduced
// modulo the target prime.  GALOIS: the source is first mapped by X -> X^galois
// (scatter through LDS; an odd multiplier permutes the LDS banks without conflicts).
// The Galois map acts on the element modulo Q: a negated coefficient is q_s - x in
// every source row, and only then is the digit lifted and reduced.
template <bool GALOIS, int ALPHA>
struct LdModup {
    static constexpr int kRaw = ALPHA;
    static constexpr bool kPrefetch = true;
    static constexpr bool kScatter = GALOIS;
    const uint64_t *src;     // ring element of unit 0
    size_t unit_stride;      // in uint64
    uint32_t galois;
    int logn;
    __device__ __forceinline__ int prime(int wg, const DevConst *C) const { return wg % C->L; }
    __device__ __forceinline__ int share(const DevConst *C) const { return C->L; }
    __device__ __forceinline__ int dst_limb(int wg, const DevConst *) const { return wg; }
    __device__ __forceinline__ void fetch(int wg, int idx, const DevConst *C, uint64_t *raw) const
    {
        const int L = C->L, j = (wg / L) % C->dnum, b = wg / (L * C->dnum);
        const uint64_t *e = src + (size_t)b * unit_stride + idx;
#pragma unroll
        for (int s = 0; s < ALPHA; s++) raw[s] = e[(size_t)(j * ALPHA + s) << logn];
    }
    __device__ __forceinline__ int place(int idx, int n) const
    {
        const uint32_t ee = ((uint32_t)idx * galois) & (2u * n - 1);
        return (int)(ee >= (uint32_t)n ? ee - n : ee);
    }
    __device__ __forceinline__ double finish(const uint64_t *raw, int wg, int idx, const ModD mr,
                                             const DevConst *C) const
    {
        const int L = C->L, r = wg % L, j = (wg / L) % C->dnum;
        bool negate = false;
        if (GALOIS) negate = (((uint32_t)idx * galois) & ((2u << logn) - 1)) >= (1u << logn);
        double x[ALPHA], a[ALPHA];
#pragma unroll
        for (int s = 0; s < ALPHA; s++) {
            x[s] = u64_to_f64(raw[s]);
            if (negate) x[s] = (x[s] == 0.0) ? 0.0 : C->mod[j * ALPHA + s].p - x[s];
        }
        if (ALPHA == 1) return x[0];     // below 2^50 is all the transform asks for
        const ConvTab &T_ = C->dig[j];
        garner<ALPHA>(T_, C->mod + j * ALPHA, x, a);
        return red(horner<ALPHA>(T_, mr, a, r), mr);
    }
};

// The mod-up of a ciphertext that a mod-down is still to deliver (one special prime, one prime to a digit; GALOIS: mapped first, as in LdModup): its second component modulo prime j is
// add + (A_j - x) / P, as moddown_kernel and moddown_sum_kernel leave it (nothing permuted is added there), canonical as every digit.
template <bool GALOIS>
struct LdModupDown {
    static constexpr int kRaw = 3;
    static constexpr bool kPrefetch = false;
    static constexpr bool kScatter = GALOIS;
    const double *acc;       // [unit][2][L][N], coefficients
    const uint64_t *add;     // second component of unit 0
    size_t add_stride;       // in uint64
    uint32_t galois;
    int logn;
    __device__ __forceinline__ int prime(int wg, const DevConst *C) const { return wg % C->L; }
    __device__ __forceinline__ int share(const DevConst *C) const { return C->L; }
    __device__ __forceinline__ int place(int idx, int n) const { return (int)((uint32_t)idx * galois & (n - 1)); }
    __device__ __forceinline__ int dst_limb(int wg, const DevConst *) const { return wg; }
    __device__ __forceinline__ void fetch(int wg, int idx, const DevConst *C, uint64_t *raw) const
    {
        const int L = C->L, k = C->k, j = (wg / L) % k, b = wg / (L * k);
        const double *a = acc + (((size_t)(2 * b + 1) * L) << logn) + idx;
        raw[0] = f64_bits(a[(size_t)j << logn]);
        raw[1] = f64_bits(a[(size_t)k << logn]);
        raw[2] = add[(size_t)b * add_stride + ((size_t)j << logn) + idx];
    }
    __device__ __forceinline__ double finish(const uint64_t *raw, int wg, int idx, const ModD, const DevConst *C) const
    {
        const int k = C->k, j = (wg / C->L) % k;
        const ModD mj = C->mod[j];
        const double x = red(bits_f64(raw[1]), C->mod[k]);
        const double v = canon(mulmod(bits_f64(raw[0]) - x, C->Pinv_q[j], mj) + u64_to_f64(raw[2]), mj);
        return GALOIS && ((uint32_t)idx * galois >> logn & 1) && v != 0.0 ? mj.p - v : v;
    }
};

// plaintext polynomial mod t -> centred lift -> row modulo q_i: workgroup -> (b, i)
struct LdPlain {
    static constexpr int kRaw = 1;
    static constexpr bool kPrefetch = true;
    static constexpr bool kScatter = false;
    const uint64_t *pt;
    int logn;
    __device__ __forceinline__ int prime(int wg, const DevConst *C) const { return wg % C->k; }
    __device__ __forceinline__ int share(const DevConst *) const { return 1; }
    __device__ __forceinline__ int dst_limb(int wg, const DevConst *) const { return wg; }
    __device__ __forceinline__ void fetch(int wg, int idx, const DevConst *C, uint64_t *raw) const
    {
        raw[0] = pt[((size_t)(wg / C->k) << logn) + idx];
    }
    __device__ __forceinline__ double finish(const uint64_t *raw, int, int, const ModD, const DevConst *C) const
    {
        const double v = u64_to_f64(raw[0]);
        return (v > 0.5 * (C->tmod - 1.0)) ? v - C->tmod : v;
    }
};

// inverse-transform loaders (finish may return any lazy value below 8p)
struct LdInvU64 {
    static constexpr int kRaw = 1;
    static constexpr bool kPrefetch = true;
    const uint64_t *src;
    const uint32_t *tab;
    int pmod, logn;
    __device__ __forceinline__ int prime(int wg, const DevConst *) const { return tab ? (int)tab[wg] : wg % pmod; }
    __device__ __forceinline__ int share(const DevConst *) const { return 1; }
    __device__ __forceinline__ int out_row(int wg, const DevConst *) const { return wg; }
    __device__ __forceinline__ void fetch(int wg, int idx, const DevConst *, uint64_t *raw) const
    {
        raw[0] = src[((size_t)wg << logn) + idx];
    }
    __device__ __forceinline__ double finish(const uint64_t *raw, int, int, const ModD, const DevConst *) const
    {
        return u64_to_f64(raw[0]);
    }
};
template <> struct inv_wide<LdInvU64> { static constexpr int value = 3; };
struct StInvU64;
template <> struct row_alone<LdInvU64, StInvU64> { static constexpr bool value = true; };
// key-switch inner product fused into the load: workgroup -> (unit b, prime r, component c), the
// component running fastest so that the two rows reading the same digits are neighbours;
struct LdInvTensor;
template <> struct inv_wide<LdInvTensor> { static constexpr int value = 2; };

// Transformed digits in memory are canonical uint64 residues, prepared keys centred residues as doubles: the
// kernels that sum in FP64 take keys as they are, and the integer accumulation of ks_sum_kernel makes integers of
// them once for several ciphertexts.  A canonical times a centred factor gives a product below 0.7 p.
template <int DNUM> __device__ __forceinline__ double inner_product(const uint64_t *raw, const ModD m)
{
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < DNUM; j++) s += mulmod(u64_to_f64(raw[2 * j]), bits_f64(raw[2 * j + 1]), m);
    return s;
}

// element = sum_j digit_j[b][r] * key[j][c][r] (both in transform order); result row [b][c][r]
template <int DNUM>
struct LdInvKsInner {
    static constexpr int kRaw = 2 * DNUM;
    static constexpr bool kPrefetch = false;
    const uint64_t *dig;   // [b][DNUM][L][N]
    const double *key;     // [DNUM][2][L][N]
    int logn;
    __device__ __forceinline__ int prime(int wg, const DevConst *C) const { return (wg >> 1) % C->L; }
    __device__ __forceinline__ int share(const DevConst *) const { return 2; }
    __device__ __forceinline__ int out_row(int wg, const DevConst *C) const
    {
        const int L = C->L, r = (wg >> 1) % L, b = wg / (2 * L);
        return (b * 2 + (wg & 1)) * L + r;
    }
    __device__ __forceinline__ void fetch(int wg, int idx, const DevConst *C, uint64_t *raw) const
    {
        const int L = C->L, r = (wg >> 1) % L, c = wg & 1, b = wg / (2 * L);
#pragma unroll
        for (int j = 0; j < DNUM; j++) {
            raw[2 * j] = dig[(((size_t)(b * DNUM + j) * L + r) << logn) + idx];
            raw[2 * j + 1] = f64_bits(key[(((size_t)(j * 2 + c) * L + r) << logn) + idx]);
        }
    }
    __device__ __forceinline__ double finish(const uint64_t *raw, int, int, const ModD m, const DevConst *) const
    {
        return inner_product<DNUM>(raw, m);
    }
};

template <int DNUM> struct ld_in<LdInvKsInner<DNUM>> { static constexpr int value = 70 * DNUM; };

// A series of rotations of the same ciphertexts ("hoisted" rotations): the digits of c1 are lifted,
// extended and transformed once, and every Galois element is applied to the transformed digits,
// where it is a permutation of the evaluation points: row element i is the value at
// psi^(2 bitrev(i) + 1), and sigma_g(a) takes there the value of a at psi^((2 bitrev(i) + 1) g).
constexpr int MAXROT = 128;   // rotations per launch
struct HoistTab {
    uint32_t g[MAXROT];            // Galois element of rotation i
    const double *key[MAXROT];     // prepared key of rotation i
};
// inner product of rotation i of unit b: workgroup -> (unit u = i * batch + b, prime r, component c);
// element = sum_j digit_j[b][r][pi_g(idx)] * key_i[j][c][r][idx]; result row [u][c][r]
template <int DNUM>
struct LdInvKsInnerHoisted {
    static constexpr int kRaw = 2 * DNUM;
    static constexpr bool kPrefetch = false;
    const uint64_t *dig;   // [b][DNUM][L][N], transform order
    HoistTab T;
    int batch, logn;
    __device__ __forceinline__ int prime(int wg, const DevConst *C) const { return (wg >> 1) % C->L; }
    __device__ __forceinline__ int share(const DevConst *) const { return 2; }
    __device__ __forceinline__ int out_row(int wg, const DevConst *C) const
    {
        const int L = C->L, r = (wg >> 1) % L, u = wg / (2 * L);
        return (u * 2 + (wg & 1)) * L + r;
    }
    __device__ __forceinline__ void fetch(int wg, int idx, const DevConst *C, uint64_t *raw) const
    {
        const int L = C->L, r = (wg >> 1) % L, c = wg & 1, u = wg / (2 * L);
        const int i = u / batch, b = u - i * batch;
        const uint32_t e = ((2u * (__brev((uint32_t)idx) >> (32 - logn)) + 1u) * T.g[i]) & ((2u << logn) - 1u);
        const int sidx = (int)(__brev(e >> 1) >> (32 - logn));
        const double *kb = T.key[i];
#pragma unroll
        for (int j = 0; j < DNUM; j++) {
            raw[2 * j] = dig[(((size_t)(b * DNUM + j) * L + r) << logn) + sidx];
            raw[2 * j + 1] = f64_bits(kb[(((size_t)(j * 2 + c) * L + r) << logn) + idx]);
        }
    }
    __device__ __forceinline__ double finish(const uint64_t *raw, int, int, const ModD m, const DevConst *) const
    {
        return inner_product<DNUM>(raw, m);
    }
};

template <int DNUM> struct ld_in<LdInvKsInnerHoisted<DNUM>> { static constexpr int value = 70 * DNUM; };

// rows of doubles (lazy), transformed in place: row w is [unit][component][prime], nprimes of them
struct LdInvF64 {
    static constexpr int kRaw = 1;
    static constexpr bool kPrefetch = true;
    const double *src;
    int nprimes, logn;
    __device__ __forceinline__ int prime(int wg, const DevConst *) const { return wg % nprimes; }
    __device__ __forceinline__ int share(const DevConst *) const { return 1; }
    __device__ __forceinline__ int out_row(int wg, const DevConst *) const { return wg; }
    __device__ __forceinline__ void fetch(int wg, int idx, const DevConst *, uint64_t *raw) const
    {
        raw[0] = f64_bits(src[((size_t)wg << logn) + idx]);
    }
    __device__ __forceinline__ double finish(const uint64_t *raw, int, int, const ModD, const DevConst *) const
    {
        return bits_f64(raw[0]);
    }
};

// tensor product fused into the load: workgroup -> (unit u, prime r of the k+l, component c in 0..2),
// the component running fastest so that the three rows reading the same four operand rows are
// neighbours; element = a0 b0 (c = 0), a0 b1 + a1 b0 (c = 1), a1 b1 (c = 2); result row [u][c][r].
// a polys of unit u: ntt[2 * (u / a_group) + {0,1}]; b polys: ntt[2 * (n_a + u) + {0,1}], or, with
// bext given, the transformed ciphertext bext[(u / b_group) * b_stride + u % b_group].
struct LdInvTensor {
    static constexpr int kRaw = 4;
    static constexpr bool kPrefetch = false;
    const double *ntt, *bext;
    int a_group, n_a, b_group, b_stride, logn;
    __device__ __forceinline__ int prime(int wg, const DevConst *C) const { return (wg / 3) % C->KL; }
    __device__ __forceinline__ int share(const DevConst *) const { return 3; }
    __device__ __forceinline__ int out_row(int wg, const DevConst *C) const
    {
        const int KL = C->KL, r = (wg / 3) % KL, u = wg / (3 * KL);
        return (u * 3 + wg % 3) * KL + r;
    }
    __device__ __forceinline__ void fetch(int wg, int idx, const DevConst *C, uint64_t *raw) const
    {
        const int KL = C->KL, c = wg % 3, r = (wg / 3) % KL, u = wg / (3 * KL);
        const size_t ps = (size_t)KL << logn, off = ((size_t)r << logn) + idx;
        const double *sa = ntt + (size_t)(2 * (u / a_group)) * ps + off;
        const double *sb = (bext ? bext + (size_t)(2 * ((u / b_group) * b_stride + u % b_group)) * ps
                                 : ntt + (size_t)(2 * (n_a + u)) * ps) + off;
        // c = 0: a0 b0; c = 2: a1 b1; c = 1: all four
        raw[0] = f64_bits(sa[c == 2 ? ps : 0]);
        raw[1] = f64_bits(sb[c == 2 ? ps : (c == 1 ? ps : 0)]);
        if (c == 1) {
            raw[2] = f64_bits(sa[ps]);
            raw[3] = f64_bits(sb[0]);
        }
    }
    __device__ __forceinline__ double finish(const uint64_t *raw, int wg, int, const ModD m, const DevConst *) const
    {
        // forward outputs are lazy: with one factor brought to p/2 the two-term sum stays below 2^52
        double s = mulmod(red(bits_f64(raw[0]), m), bits_f64(raw[1]), m);
        if (wg % 3 == 1) s += mulmod(red(bits_f64(raw[2]), m), bits_f64(raw[3]), m);
        return s;
    }
};

// The tensor products of a group of consecutive units summed before the inverse transform (and so
// before the one scaling that follows): workgroup -> (group g, prime r, component c); element =
// sum over the group's units u = g * group + i of the element LdInvTensor forms for u; result row
// [g][c][r].  Operand addressing as in LdInvTensor.
struct LdInvTensorSum {
    static constexpr int kRaw = 4;
    static constexpr bool kPrefetch = false;
    LdInvTensor one;
    int group;
    __device__ __forceinline__ int prime(int wg, const DevConst *C) const { return (wg / 3) % C->KL; }
    __device__ __forceinline__ int share(const DevConst *) const { return 3; }
    __device__ __forceinline__ int out_row(int wg, const DevConst *C) const { return one.out_row(wg, C); }
    __device__ __forceinline__ int rounds() const { return group; }
    __device__ __forceinline__ void fetch_round(int wg, int idx, int i, const DevConst *C, uint64_t *raw) const
    {
        const int per = 3 * C->KL, g = wg / per;
        one.fetch((g * group + i) * per + wg % per, idx, C, raw);
    }
    __device__ __forceinline__ void fetch(int, int, const DevConst *, uint64_t *) const {}
    __device__ __forceinline__ double finish(const uint64_t *raw, int wg, int idx, const ModD m, const DevConst *C) const
    {
        return one.finish(raw, wg, idx, m, C);     // only wg % 3 matters there
    }
    // a unit's term is below 4 p
    __device__ __forceinline__ double join(double sum, double term, const ModD m) const { return red(sum, m) + term; }
};
template <> struct ld_rounds<LdInvTensorSum> { static constexpr bool value = true; };
static_assert(fwd_out<12>() <= fwd_out<13>(), "the bound of both");
template <> struct ld_in<LdInvTensor> { static constexpr int value = hundredths(2.0 * prod_of(fwd_out<13>())); };
template <> struct ld_in<LdInvTensorSum> { static constexpr int value = hundredths(0.51 + 2.0 * prod_of(fwd_out<13>())); };
template <> struct ld_no_16384<LdInvTensor> { static constexpr bool value = true; };
template <> struct ld_no_16384<LdInvTensorSum> { static constexpr bool value = true; };

// transformed ciphertext row times prepared plaintext row (ct x pt fused into the load):
// workgroup -> (unit b, comp c, prime i); ciphertext = ctf[b / ct_group], plaintext =
// plain[(b % p_mod) * pstride + pofs]
struct LdInvMulPlain {
    static constexpr int kRaw = 2;
    static constexpr bool kPrefetch = true;
    const double *ctf;     // forward-transformed ciphertext rows [*][2][k][N]
    const double *plain;   // prepared plaintexts [*][k][N]
    int ct_group, p_mod, pstride, pofs, logn;
    __device__ __forceinline__ int prime(int wg, const DevConst *C) const { return wg % C->k; }
    __device__ __forceinline__ int share(const DevConst *) const { return 1; }
    __device__ __forceinline__ int out_row(int wg, const DevConst *) const { return wg; }
    __device__ __forceinline__ void fetch(int wg, int idx, const DevConst *C, uint64_t *raw) const
    {
        const int k = C->k, i = wg % k, c = (wg / k) & 1, b = wg / (2 * k);
        raw[0] = f64_bits(ctf[((size_t)(((b / ct_group) * 2 + c) * k + i) << logn) + idx]);
        raw[1] = f64_bits(plain[((size_t)(((b % p_mod) * pstride + pofs) * k + i) << logn) + idx]);
    }
    __device__ __forceinline__ double finish(const uint64_t *raw, int, int, const ModD m, const DevConst *) const
    {
        return mulmod(bits_f64(raw[0]), bits_f64(raw[1]), m);
    }
};

// sum of ciphertext-plaintext products fused into the load (the decode step's vector-matrix
// product): workgroup -> (unit u, comp c2, prime i); element = sum over the cn rotated copies of
// the token of copy_c[c2][i] * diagonal_(u, c)[i].  Eight elements' words of one copy are asked for together; a
// loop over the copies inside an element had its two words' trip to memory to wait for at every step.  36 matrices
// of 8 diagonals, N = 8192, 37 us in this launch: the call 245 -> 233 us; 96 of 16: 655 -> 555 us.  (Rows of a unit on one
// XCD, so that its L2 serves both components' reads of a diagonal: 243 us.  The next copy's words asked for ahead: 235,
// registers spilled.)
struct LdInvPlainSum {
    static constexpr int kRaw = 2;
    static constexpr bool kPrefetch = false;
    const double *ctf;     // transformed copies [cn][2][k][N], |x| <= p/2
    const double *plain;   // prepared plaintexts [units][cn][k][N]
    int cn, logn;
    __device__ __forceinline__ int prime(int wg, const DevConst *C) const { return wg % C->k; }
    __device__ __forceinline__ int share(const DevConst *) const { return 1; }
    __device__ __forceinline__ int out_row(int wg, const DevConst *) const { return wg; }
    __device__ __forceinline__ int rounds() const { return cn; }
    __device__ __forceinline__ void fetch_round(int wg, int idx, int c, const DevConst *C, uint64_t *raw) const
    {
        const int k = C->k, i = wg % k, c2 = (wg / k) & 1, u = wg / (2 * k);
        raw[0] = f64_bits(at32(ctf + ((size_t)((c * 2 + c2) * k + i) << logn), idx));
        raw[1] = f64_bits(at32(plain + ((((size_t)u * cn + c) * k + i) << logn), idx));
    }
    __device__ __forceinline__ void fetch(int, int, const DevConst *, uint64_t *) const {}
    __device__ __forceinline__ double finish(const uint64_t *raw, int, int, const ModD m, const DevConst *) const
    {
        return mulmod(bits_f64(raw[0]), bits_f64(raw[1]), m);
    }
    // the copies are stored reduced: a product is below 0.6 p
    __device__ __forceinline__ double join(double sum, double term, const ModD m) const { return red(sum, m) + term; }
};
template <> struct ld_rounds<LdInvPlainSum> { static constexpr bool value = true; };

struct StInvF64 {
    double *dst;
    int logn;
    __device__ __forceinline__ void store(int wg, int idx, double v, const ModD) const
    {
        put32(dst + ((size_t)wg << logn), idx, v);
    }
    // element `at` + `lane` of the row, `at` uniform
    __device__ __forceinline__ void store_lane(int wg, int at, int lane, double v, const ModD) const
    {
        put_lane(dst + ((size_t)wg << logn) + at, lane, v);
    }
};
// rows of a tensor product without N^-1.  HALF: half rows, whose sums and differences the scaling takes.  (scale_kernel adds a reduced
// value to a result, or to such a sum: below 2^53 together.)
template <bool HALF> struct StTens : StInvF64 {};
template <bool HALF> struct st_unscaled<StTens<HALF>> { static constexpr int value = HALF ? 365 : 730; };
struct StInvU64 {
    uint64_t *dst;
    int logn;
    __device__ __forceinline__ void store(int wg, int idx, double v, const ModD m) const
    {
        put32(dst + ((size_t)wg << logn), idx, f64_to_u64(canon(v, m)));
    }
    // (with the row's address in scalar registers 4323 rows of 8192 take 157.4 us instead of 155.8, 1025 of 16384 75.6 instead of 74.3)
    __device__ __forceinline__ void store_lane(int wg, int at, int lane, double v, const ModD m) const { store(wg, at + lane, v, m); }
    __device__ __forceinline__ const StInvU64 &at_row(int, int) const { return *this; }
};
// cache append: workgroup -> (cache c, comp, prime); target row = cache + c*stride + row;
// fresh != 0 stores, otherwise adds to what is there
struct StAppendRow {        // for one row
    uint64_t *row;
    int fresh;
    // the words of elements tid + c T, c = c0 .. c0 + 7: one branch around all the loads.  (A test per element became a
    // block per two loads with a wait in each, four trips to memory one after the other in every append: 24 caches of
    // N = 8192, 128 appends 2113 us, now 1982.)
    template <int T> __device__ __forceinline__ void fetch(uint64_t *old, int tid, int c0) const
    {
#pragma unroll
        for (int c = 0; c < 8; c++) old[c] = 0;
        if (!fresh) {
#pragma unroll
            for (int c = 0; c < 8; c++) old[c] = at_lane(row + (c0 + c) * T, tid);
        }
    }
    // (v is below 2 p and old below p: one reduction of the sum)
    __device__ __forceinline__ void store(int at, int lane, double v, uint64_t old, const ModD m) const
    {
        put_lane(row + at, lane, f64_to_u64(canon(v + u64_to_f64(old), m)));
    }
};
struct StInvAppend {
    uint64_t *cache;        // first target ciphertext (cache 0)
    size_t cache_stride;    // uint64 between consecutive caches' target ciphertexts
    int fresh, logn;
    __device__ __forceinline__ StAppendRow at_row(int wg, int k) const
    {
        const int rows = 2 * k, c = wg / rows, row = wg % rows;
        return StAppendRow{cache + (size_t)c * cache_stride + ((size_t)row << logn), fresh};
    }
};
template <> struct st_adds<StAppendRow> { static constexpr bool value = true; };

// ---------------------------------------------------------------------------
// Transforms of a row that is in registers already or stays there: the pass sequence only.
// ---------------------------------------------------------------------------
// in: pass-0 ownership (element tid + it * T), or, with SCATTERED, already in LDS; out: chunk_elem order
// ahead: run before the last pass, for loads that nothing before it waits for
struct Nothing { __device__ __forceinline__ void operator()() const {} };
// U: rows of one prime together, row u in in[u E ...], its LDS u * lds_doubles() further on
template <int LOGN, int E, bool SCATTERED, bool PRIO = false, int U = 1, int IN = (int)(100 * FWD_IN), class F = Nothing>
__device__ __forceinline__ void fwd_row(double *lds, const double *in, double *out, int tid,
                                        const double *__restrict__ tw, const ModD m, F ahead = F(), int root = 1)
{
    constexpr int NP = Plan<LOGN, E>::NP;
    // addresses are formed here and now: hoisted out of the caller's loops they would take the registers
    // that hold its rows
    asm volatile("" : "+v"(tid));
    double twa[TWREGS], twb[TWREGS];
    const StRegs st{out};
    load_tw<LOGN, E, 0, true>(tw, tid, twa, root);
    fwd_pass<LOGN, E, 0, !SCATTERED, U, IN>(lds, in, st, tid, tw, twa, twb, m, 0, PRIO, root);
    fwd_pass<LOGN, E, 1, false, U, IN>(lds, in, st, tid, tw, twb, twa, m, 0, PRIO, root);
    fwd_pass<LOGN, E, 2, false, U, IN>(lds, in, st, tid, tw, twa, twb, m, 0, PRIO, root);
    if (NP == 4) ahead();
    fwd_pass<LOGN, E, 3, false, U, IN>(lds, in, st, tid, tw, twb, twa, m, 0, PRIO, root);
    if (NP > 4) ahead();
    if constexpr (NP > 4) fwd_pass<LOGN, E, 4, false, U, IN>(lds, in, st, tid, tw, twa, twb, m, 0, PRIO, root);
}
// in: chunk_elem order, |x| < 8p (or the bound IN in hundredths); results leave through st as row `row`
// U: rows together as in fwd_row, results as rows `row` + u * row_step
// ahead: run before the last two passes, whose factors are scalar loads: nothing in them waits behind the loads it asks for
template <int LOGN, int E, bool PRIO = false, int IN = 0, int U = 1, class ST, class F = Nothing>
__device__ __forceinline__ void inv_row(double *lds, const double *in, const ST &st, int row, int tid,
                                        const double *__restrict__ itw, const ModD m, int pr, const DevConst *C,
                                        int row_step = 0, F ahead = F(), int root = 1)
{
    constexpr int NP = Plan<LOGN, E>::NP;
    asm volatile("" : "+v"(tid));
    double twa[TWREGS], twb[TWREGS];
    load_tw<LOGN, E, NP - 1, false>(itw, tid, twa, root);
    if constexpr (Plan<LOGN, E>::R[NP - 1] != 1) {
#pragma unroll
        for (int it = 0; it < U * E; it += 2)
            pair_at(lds, it / E * lds_doubles<LOGN>() + pad(chunk_elem<E>(tid, it % E))) = make_double2(in[it], in[it + 1]);
        wave_sync();
    }
    inv_pass<LOGN, E, NP - 1, IN, U>(lds, st, row, tid, itw, twa, twb, m, pr, C, in, nullptr, PRIO, row_step, root);
    if constexpr (NP > 4) {
        inv_pass<LOGN, E, 3, IN, U>(lds, st, row, tid, itw, twb, twa, m, pr, C, nullptr, nullptr, PRIO, row_step, root);
        inv_pass<LOGN, E, 2, IN, U>(lds, st, row, tid, itw, twa, twb, m, pr, C, nullptr, nullptr, PRIO, row_step, root);
        ahead();
        inv_pass<LOGN, E, 1, IN, U>(lds, st, row, tid, itw, twb, twa, m, pr, C, nullptr, nullptr, PRIO, row_step, root);
        inv_pass<LOGN, E, 0, IN, U>(lds, st, row, tid, itw, twa, twb, m, pr, C, nullptr, nullptr, PRIO, row_step, root);
    } else {
        inv_pass<LOGN, E, 2, IN, U>(lds, st, row, tid, itw, twb, twa, m, pr, C, nullptr, nullptr, PRIO, row_step, root);
        ahead();
        inv_pass<LOGN, E, 1, IN, U>(lds, st, row, tid, itw, twa, twb, m, pr, C, nullptr, nullptr, PRIO, row_step, root);
        inv_pass<LOGN, E, 0, IN, U>(lds, st, row, tid, itw, twb, twa, m, pr, C, nullptr, nullptr, PRIO, row_step, root);
    }
}

// ---------------------------------------------------------------------------
// Key switch of one (unit, prime) per workgroup (digits of one prime): the digits lifted and transformed one after the
// other, each multiplied with its two key rows into two sums in registers, and the sums transformed back.
// The transformed digits never reach memory (24 of 35 rows per unit of traffic less) and five transforms follow
// each other without a launch between them.  The sums go back together: each wait at a barrier and each factor serves both
// (with ks_sum_row_kernel and ks_unit_kernel: 768 products with relinearisation 1780 -> 1760 us, a chain step of 12 heads 659 -> 652,
// scores of 12 heads 9150 -> 9041).  Bound by vector issue (71 % busy on 700 units): 1024 threads with
// eight elements each, because a row is then 16 registers and the two sums, the row, its factors and the next
// digit's words fit 128.  768 units at N = 8192, three digits, four primes: 284 + 376 us for the mod-up and inner product
// launches, 383 us here.
// ---------------------------------------------------------------------------
template <int LOGN, int E, bool GALOIS>
__global__ void __launch_bounds__((1 << LOGN) / E, (min_waves<LOGN, E>()))
ks_row_kernel(LdModup<GALOIS, 1> ld, const double *__restrict__ key, StInvF64 st,
              const double *__restrict__ tw_all, const double *__restrict__ itw_all, const DevConst *__restrict__ C,
              int nwg)
{
    __shared__ __align__(16) double lds[2 * lds_doubles<LOGN>()];
    constexpr int T = (1 << LOGN) / E;
    const int tid = threadIdx.x, L = C->L, dnum = C->dnum;
    int p = blockIdx.x;
    int wg = xcd_row(p, nwg, L);
    auto at = [&](int it) { return GALOIS ? chunk_elem<E>(tid, it) : tid + it * T; };
    uint64_t raw[E][1];
    auto fetch = [&](int b, int j) {
        const uint64_t *e = ld.src + (size_t)b * ld.unit_stride + ((size_t)j << LOGN);
#pragma unroll
        for (int it = 0; it < E; it++) raw[it][0] = GALOIS ? at32(e, at(it)) : at_lane(e + it * T, tid);
    };
    fetch(wg / L, 0);
    for (;;) {
        const int r = wg % L, b = wg / L;
        const ModD m = C->mod[r];
        const double *tw = tw_all + ((size_t)r << LOGN), *itw = itw_all + ((size_t)r << LOGN);
        p += (int)gridDim.x;
        const bool more = p < nwg;
        const int wg_next = more ? xcd_row(p, nwg, L) : wg;
        double s[2 * E];
#pragma unroll
        for (int it = 0; it < 2 * E; it++) s[it] = 0.0;
        for (int j = 0; j < dnum; j++) {
            double x[E];
            const int row = (b * dnum + j) * L + r;
#pragma unroll
            for (int it = 0; it < E; it++) x[it] = ld.finish(raw[it], row, at(it), m, C);
            fetch(j + 1 < dnum ? b : wg_next / L, j + 1 < dnum ? j + 1 : 0);    // (once too often at the very end)
            if constexpr (GALOIS) {
#pragma unroll
                for (int it = 0; it < E; it++) lds[pad(ld.place(at(it), 1 << LOGN))] = x[it];
                lds_barrier();
            }
            fwd_row<LOGN, E, GALOIS>(lds, x, x, tid, tw, m);
            const double *k0 = key + ((size_t)(2 * j * L + r) << LOGN), *k1 = k0 + ((size_t)L << LOGN);
            int tk = tid;
            asm volatile("" : "+v"(tk));
            // a lazy value times a centred key is below 2 p: up to three of them need no reduction before
            if (dnum > 3) {
#pragma unroll
                for (int it = 0; it < E; it++) x[it] = red(x[it], m);
            }
#pragma unroll
            for (int it = 0; it < E; it++) {
                const int idx = chunk_elem<E>(tk, it);
                s[it] += mulmod(x[it], at32(k0, idx), m);
                s[E + it] += mulmod(x[it], at32(k1, idx), m);
            }
            if (j + 1 < dnum) lds_barrier();
        }
        inv_row<LOGN, E, false, 0, 2>(lds, s, st, (b * 2) * L + r, tid, itw, m, r, C, L);
        if (!more) break;
        wg = wg_next;
        lds_barrier();
    }
}

// A sum of products reduced once: `a` adds up the products' multiples of 2^50 (from 1.5 * 2^102 on, where an FP64 number's last bit is worth
// 2^50), `l` what each addition rounded away, which the next FMA returns exactly.  Four instructions a product where one that is
// reduced and added takes seven; close() takes six.  Between open and close up to CENTRED products of centred residues (below 2^98
// each), or up to CANONICAL of a canonical and a centred one (below 2^99): a stays within 2^102 ... 2^103, l within 4 * 2^50 of what it was opened with.  close(): the quotient of a sum of 2^101 at most is off by 1/4 for
// rounding h + l, the reciprocal and the product each, so the result is below 1.25 * 2^50, and fma(-c, p, h) = result - l below
// 2^53: exact.
struct DotSum {
    static constexpr int CENTRED = 8, CANONICAL = 4;
    static constexpr double ZERO = 0x1.8p102, OUT = 1.26;
    double a, l;
    __device__ __forceinline__ void open(double start) { a = ZERO, l = start; }
    __device__ __forceinline__ void add(double x, double w)
    {
        const double t = __builtin_fma(x, w, a);
        l += __builtin_fma(x, w, a - t);
        a = t;
    }
    __device__ __forceinline__ double close(const ModD m) const
    {
        const double h = a - ZERO, c = __builtin_rint((h + l) * m.u);
        return __builtin_fma(-c, m.p, h) + l;
    }
};

// A transformed digit (reduced, in LDS) times the keys of n_rot rotations, each at its permuted evaluation points, added to the two sums
// s[0 ... E) and s[E ... 2 E).  W pairs of elements are taken through all rotations before the next ones, so that only their sums are open; keys are asked
// for a pair ahead, their addresses and Galois elements read a rotation ahead.  us a series of 7 rotations, N = 8192, three digits: with products reduced
// one by one 64 ciphertexts 80.3, now 76.7; 15 rotations 119 / 111.  (For two units and at N = 16384, where four sums leave no registers for
// open ones but a pair at a time, even at 7 rotations and 3 to 12 % slower at one.)
struct RotWalk {
    const HoistTab &T;
    int n, at;                          // rotation of g_next, key_next
    size_t row;
    uint32_t g, g_next;
    const double *key, *key_next;
    __device__ __forceinline__ void look()
    {
        g_next = T.g[at];
        key_next = T.key[at] + row;
    }
    __device__ __forceinline__ void step()
    {
        g = g_next;
        key = key_next;
        at = at + 1 == n ? 0 : at + 1;
        look();
    }
    __device__ __forceinline__ RotWalk(const HoistTab &T_, int n_, size_t row_) : T(T_), n(n_), at(0), row(row_)
    {
        look();
        step();
    }
};
__device__ __forceinline__ void ask_pair(const double *key, size_t comp, int lane, cg_double2v (&k)[2])
{
    const cg_double2v *k0 = reinterpret_cast<const cg_double2v *>(key);
    k[0] = at_lane(k0, lane);
    k[1] = at_lane(k0 + comp, lane);
}
// pairs F ... F + W - 1, and those behind; k[0]: the first one's keys
template <int LOGN, int E, int W, int F>
__device__ __forceinline__ void sum_pairs(const double *lds, RotWalk &way, size_t comp, int lane, uint32_t e0, const ModD m, double (&s)[2 * E],
                                          cg_double2v (&k)[2][2])
{
    static_assert(W % 2 == 0, "the two sets of keys keep their registers");
    constexpr int NEXT = F + W < E / 2 ? F + W : F;
    DotSum d[4 * W];        // [pair][component][element]
#pragma unroll
    for (int x = 0; x < 4 * W; x++) d[x].open(s[x / 2 % 2 * E + 2 * (F + x / 4) + x % 2]);
    int i = 0;
    do {
#pragma unroll
        for (int w = 0; w < W; w++) {
            // (behind the last pair the next rotation's first one, behind the last rotation that of the next pairs)
            if (w + 1 < W) ask_pair(way.key + 128 * (F + w + 1), comp, lane, k[(w + 1) & 1]);
            else ask_pair(way.key_next + 128 * (i + 1 < way.n ? F : NEXT), comp, lane, k[(w + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            // evaluation point of the pair's first element under the map; its second's is the neighbour that differs in the
            // lowest bit.  (Bits above the row's fall out on the right.)
            const uint32_t e = __umul24(e0 + 2u * (__brev((uint32_t)(128 * (F + w))) >> (32 - LOGN)), way.g);
            const int at = pad((int)((__brev(e) >> (31 - LOGN)) & ((1u << LOGN) - 1u)));
            const double x0 = lds[at], x1 = lds[at ^ 1];
#pragma unroll
            for (int c = 0; c < 2; c++) {
                d[4 * w + 2 * c].add(x0, k[w & 1][c].x);
                d[4 * w + 2 * c + 1].add(x1, k[w & 1][c].y);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        way.step();
        i++;
        if (i % DotSum::CENTRED == 0 && i < way.n) {
#pragma unroll
            for (int x = 0; x < 4 * W; x++) d[x].open(d[x].close(m));
        }
    } while (i < way.n);
#pragma unroll
    for (int x = 0; x < 4 * W; x++) s[x / 2 % 2 * E + 2 * (F + x / 4) + x % 2] = d[x].close(m);
    if constexpr (F + W < E / 2) sum_pairs<LOGN, E, W, F + W>(lds, way, comp, lane, e0, m, s, k);
}
template <int LOGN, int E, int W>
__device__ __forceinline__ void sum_digit(const double *lds, const HoistTab &T, int n_rot, int j, int r, int L, int tk, const ModD m, double (&s)[2 * E])
{
    const int idx0 = chunk_elem<E>(tk, 0);
    const size_t comp = (size_t)L << (LOGN - 1);
    RotWalk way(T, n_rot, (size_t)(2 * j * L + r) << LOGN);
    cg_double2v k[2][2];
    ask_pair(way.key, comp, idx0 / 2, k[0]);
    sum_pairs<LOGN, E, W, 0>(lds, way, comp, idx0 / 2, 2u * (__brev((uint32_t)idx0) >> (32 - LOGN)) + 1u, m, s, k);
}

// The same for two units, their digits ROW doubles apart in LDS: a key is read once for both, a pair of elements ahead of its use
template <int LOGN, int E>
__device__ __forceinline__ void sum_digits(const double *lds, const HoistTab &T, int n_rot, int j, int r, int L, int tk,
                                           const ModD m, double *s0, double *s1, double *s2, double *s3)
{
    constexpr int ROW = lds_doubles<LOGN>();
    const int idx0 = chunk_elem<E>(tk, 0);
    const uint32_t e0 = 2u * (__brev((uint32_t)idx0) >> (32 - LOGN)) + 1u;
    const size_t comp = (size_t)L << (LOGN - 1);
    auto rows = [&](int i) { return reinterpret_cast<const cg_double2v *>(T.key[i] + ((size_t)(2 * j * L + r) << LOGN)); };
    const cg_double2v *k0 = rows(0);
    uint32_t g = T.g[0];
    cg_double2v a[2], c[2];
    a[0] = at_lane(k0, idx0 / 2);
    c[0] = at_lane(k0 + comp, idx0 / 2);
    for (int i = 0; i < n_rot; i++) {
        const int i_next = i + 1 < n_rot ? i + 1 : i;
        const cg_double2v *kn = rows(i_next);
        const uint32_t gn = T.g[i_next], eg = __umul24(e0, g);
#pragma unroll
        for (int q = 0; q < E / 2; q++) {
            const cg_double2v *kq = q + 1 < E / 2 ? k0 + 64 * (q + 1) : kn;
            a[(q + 1) & 1] = at_lane(kq, idx0 / 2);
            c[(q + 1) & 1] = at_lane(kq + comp, idx0 / 2);
            __builtin_amdgcn_sched_barrier(0);
            const cg_double2v ka = a[q & 1], kc = c[q & 1];
            const uint32_t e = eg + 2u * (__brev((uint32_t)(128 * q)) >> (32 - LOGN)) * g;
            const int at = pad((int)((__brev(e) >> (31 - LOGN)) & ((1u << LOGN) - 1u)));
            const double x0 = lds[at], x1 = lds[at ^ 1], y0 = lds[ROW + at], y1 = lds[ROW + (at ^ 1)];
            s0[2 * q] += mulmod(x0, ka.x, m);
            s0[2 * q + 1] += mulmod(x1, ka.y, m);
            s1[2 * q] += mulmod(x0, kc.x, m);
            s1[2 * q + 1] += mulmod(x1, kc.y, m);
            s2[2 * q] += mulmod(y0, ka.x, m);
            s2[2 * q + 1] += mulmod(y1, ka.y, m);
            s3[2 * q] += mulmod(y0, kc.x, m);
            s3[2 * q + 1] += mulmod(y1, kc.y, m);
            __builtin_amdgcn_sched_barrier(0);
        }
        k0 = kn;
        g = gn;
        if ((i & 7) == 7 || i + 1 == n_rot) {
#pragma unroll
            for (int it = 0; it < E; it++) {
                s0[it] = red(s0[it], m);
                s1[it] = red(s1[it], m);
                s2[it] = red(s2[it], m);
                s3[it] = red(s3[it], m);
            }
        }
    }
}

// mod-down with rounding and the final additions of relinearisation / rotation:
//   u = floor((A + floor(P/2)) / P) = (A - x) / P mod Q with x the centred residue of A modulo P, in balanced
//   digits (garner_balanced takes the transforms' results, below 2p);  out[b][c] = u (+ add0) (+ add1)
// add0: relin -> in3[b][c];  rotate -> sigma_g(in2[b][0]) for c = 0, nothing for c = 1
// add1: rotate with accumulate -> acc_add[b][c] (the rotated ciphertext itself, or another one)
struct ModdownArgs {
    const double *acc;        // [b][2][L][N] lazy, coefficient order
    uint64_t *out;            // unit b at out + b*out_stride, [2][k][N]
    size_t out_stride;
    const uint64_t *add;      // base of the addend ciphertexts (unit 0) or null
    size_t add_stride;        // uint64 per unit in add
    uint32_t galois;          // != 0: add is permuted by X -> X^galois and only applies to c = 0
    int accumulate;           // also add the un-permuted acc_add[b][c]
    int batch;
    const uint64_t *acc_add;  // base of the ciphertexts added un-permuted (accumulate)
    size_t acc_stride;
};
// HOIST: the units are the rotations of a series, unit u = i * rot_batch + b being rotation i of
// ciphertext b: its Galois element comes from the table, its addend is ciphertext b and its output
// ciphertext b * out_per_b + i.
// n_sum: rotations whose accumulators were summed (moddown_sum_kernel).
template <int LOGN> constexpr int moddown_sum_split() { return (1 << LOGN) / 2048 >= 4 ? 4 : (1 << LOGN) / 2048; }
struct ModdownHoist {
    uint32_t ginv[MAXROT];
    int rot_batch, out_per_b, n_sum;
};
// a + w or a - w as the top bit of s says
__device__ __forceinline__ double signed_add(double a, double w, uint32_t s)
{
    return a + bits_f64(f64_bits(w) ^ ((uint64_t)(s & 0x80000000u) << 32));
}
// ---------------------------------------------------------------------------
// Summed rotations of one (unit, prime), or of two units, per workgroup: digits lifted and transformed one after the other; a
// transformed digit lies in LDS, from where every rotation takes its permuted values, while the keys stream past;
// the two sums in registers are transformed back.  With digits through memory (ks_sum_kernel) every rotation's
// gather of every digit goes to L2, and half of them miss it; here the keys are what comes in, and an XCD works with
// the keys of one or two primes.  Bound by the keys' way from L2 (128 KB a rotation and digit, 39 bytes a clock and compute unit) and
// by vector issue (74 % busy with two units); two units to a workgroup halve the first.  N = 8192, 7 rotations, 1536 ciphertexts:
// mod-up, sums and inverse transforms 475 + 899 + 369 us in three launches, 1513 us here with one unit, 1391 with two (1314
// since the two sums of a unit are transformed back together).
// ---------------------------------------------------------------------------
// the sums of units b ... b + U - 1 (those of the batch) modulo prime r: s (both components), and of a second unit s2 and s3
// AGAIN: LDS places worked out for each digit again instead of held, which the kernel that divides by P has no registers for
template <int LOGN, int E, int U, bool AGAIN>
__device__ __forceinline__ void sum_units(double *lds, const LdModup<false, 1> &ld, const HoistTab &T, int n_rot, int batch, int b, int r, int tid,
                                          const double *__restrict__ tw, const ModD m, const DevConst *__restrict__ C, double (&s)[2 * E],
                                          double (&s2)[U > 1 ? E : 1], double (&s3)[U > 1 ? E : 1])
{
    constexpr int TH = (1 << LOGN) / E, ROW = lds_doubles<LOGN>();
    const int L = C->L, dnum = C->dnum;
    uint64_t raw[E][1];
    // (an odd batch's last workgroup takes its one unit twice and stores it once)
    auto fetch = [&](int u, int j) {
        const uint64_t *src = ld.src + (size_t)(b + u < batch ? b + u : b) * ld.unit_stride + ((size_t)j << LOGN);
#pragma unroll
        for (int it = 0; it < E; it++) raw[it][0] = at_lane(src + it * TH, tid);
    };
    fetch(0, 0);
#pragma unroll
    for (int it = 0; it < E; it++) {
        s[it] = s[E + it] = 0.0;
        if (U > 1) s2[it % (U > 1 ? E : 1)] = s3[it % (U > 1 ? E : 1)] = 0.0;
    }
    for (int j = 0; j < dnum; j++) {
#pragma unroll
        for (int u = 0; u < U; u++) {
            double x[E];
            const int row = ((b + u) * dnum + j) * L + r;
#pragma unroll
            for (int it = 0; it < E; it++) x[it] = ld.finish(raw[it], row, tid + it * TH, m, C);
            if (u == 0) lds_barrier();      // the previous digit's (or unit's) LDS reads
            fwd_row<LOGN, E, false>(lds + u * ROW, x, x, tid, tw, m);
            if (U > 1) fetch(u + 1 < U ? u + 1 : 0, u + 1 < U || j + 1 == dnum ? j : j + 1);
            int ts = tid;
            if (AGAIN) asm volatile("" : "+v"(ts));
#pragma unroll
            for (int it = 0; it < E; it += 2)
                pair_at(lds + u * ROW, pad(chunk_elem<E>(ts, it))) = make_double2(red(x[it], m), red(x[it + 1], m));
        }
        lds_barrier();
        int tk = tid;
        asm volatile("" : "+v"(tk));
        if constexpr (U == 1) sum_digit<LOGN, E, 4>(lds, T, n_rot, j, r, L, tk, m, s);
        else sum_digits<LOGN, E>(lds, T, n_rot, j, r, L, tk, m, s, s + E, s2, s3);
        if (U == 1) fetch(0, j + 1 < dnum ? j + 1 : j);     // (sooner there are no registers for it: 77.9 us there, 79.5 before the transform)
    }
    lds_barrier();
}
// What an inverse transform of a sum may expect
template <int U> constexpr int sum_bound() { return U > 1 ? 52 : hundredths(DotSum::OUT); }

// r0: first prime of the launch
template <int LOGN, int E, int U>
__global__ void __launch_bounds__((1 << LOGN) / E, (min_waves<LOGN, E>()))
ks_sum_row_kernel(LdModup<false, 1> ld, HoistTab T, int n_rot, int batch, StInvF64 st,
                  const double *__restrict__ tw_all, const double *__restrict__ itw_all,
                  const DevConst *__restrict__ C, int nwg, int r0)
{
    static_assert(U == 1 || U == 2, "units of a workgroup");
    __shared__ __align__(16) double lds[2 * lds_doubles<LOGN>()];
    const int tid = threadIdx.x, L = C->L, sets = (batch + U - 1) / U;
    // logical order: prime, then unit; XCD x takes the x-th eighth of it, so that an XCD works with the keys
    // of one or two primes
    const int per_xcd = (nwg + 7) >> 3;
    auto logical = [&](int p) { return (p & 7) * per_xcd + (p >> 3); };
    const int total = per_xcd * 8;
    for (int p = blockIdx.x; p < total; p += (int)gridDim.x) {
        const int wg = logical(p);
        if (wg >= nwg) continue;
        const int q = wg / sets, r = r0 + q, b = (wg - q * sets) * U;
        const ModD m = C->mod[r];
        const double *tw = tw_all + ((size_t)r << LOGN), *itw = itw_all + ((size_t)r << LOGN);
        double s[2 * E], s2[U > 1 ? E : 1], s3[U > 1 ? E : 1];
        sum_units<LOGN, E, U, false>(lds, ld, T, n_rot, batch, b, r, tid, tw, m, C, s, s2, s3);
        // both components of a unit
        auto inverse = [&](const double *a, const double *c, int unit) {
            double y[2 * E];
#pragma unroll
            for (int it = 0; it < E; it++) {
                y[it] = a[it];
                y[E + it] = c[it];
            }
            inv_row<LOGN, E, false, sum_bound<U>(), 2>(lds, y, st, (unit * 2) * L + r, tid, itw, m, r, C, L);
        };
        inverse(s, s + E, b);
        if (U > 1 && b + 1 < batch) {
            lds_barrier();
            inverse(s2, s3, b + 1);
        }
    }
}

// The same modulo the ciphertext primes, two units to a workgroup, once the accumulators modulo the special prime are there: the division by P
// and the additions follow in registers, c0 permuted through LDS, as in ks_unit_kernel.  The accumulators of the other primes (six rows of
// eight a ciphertext, written and read again) never reach memory and the mod-down launch, which memory bounds, is gone.  N = 8192, three digits, 7
// rotations, 1536 ciphertexts: 1723 us with the mod-down, 1568 here and for the special prime (1673 with component 1's words asked for only when
// component 0 is stored); what follows the transforms takes 24 to 31 us a workgroup, twelve rows' trips from memory.  A flag that was spilled (is there a
// rotation at all) had component 1's words waited for before component 0's rotations: 1242 us a launch of 1536 ciphertexts, 1231 since nothing is.
template <int LOGN, int E>
__global__ void __launch_bounds__((1 << LOGN) / E, (min_waves<LOGN, E>()))
ks_sum_down_kernel(LdModup<false, 1> ld, HoistTab T, ModdownArgs A, ModdownHoist H, const double *__restrict__ tw_all,
                   const double *__restrict__ itw_all, const DevConst *__restrict__ C, int nwg)
{
    constexpr int TH = (1 << LOGN) / E, N = 1 << LOGN;
    __shared__ __align__(16) double lds[2 * lds_doubles<LOGN>()];
    const int tid = threadIdx.x, k = C->k, L = C->L, sets = (A.batch + 1) / 2;
    const int per_xcd = (nwg + 7) >> 3, total = per_xcd * 8;       // as in ks_sum_row_kernel
    for (int p = blockIdx.x; p < total; p += (int)gridDim.x) {
        const int wg = (p & 7) * per_xcd + (p >> 3);
        if (wg >= nwg) continue;
        const int r = wg / sets, b0 = (wg - r * sets) * 2;
        const ModD m = C->mod[r];
        const double *tw = tw_all + ((size_t)r << LOGN), *itw = itw_all + ((size_t)r << LOGN);
        double s[2 * E], s2[E], s3[E];
        sum_units<LOGN, E, 2, true>(lds, ld, T, H.n_sum, A.batch, b0, r, tid, tw, m, C, s, s2, s3);
        auto finish = [&](const double *s0, const double *s1, int b) {
            double y[2 * E], xs[E];
            uint64_t own[E];
            const size_t row = (size_t)r << LOGN, comp = (size_t)k << LOGN;
            const double *special = A.acc + ((size_t)(2 * b * L + k) << LOGN);
            const uint64_t *in = A.add + (size_t)b * A.add_stride + row;
            uint64_t *out = A.out + (size_t)b * A.out_stride + row;
#pragma unroll
            for (int it = 0; it < E; it++) {
                y[it] = s0[it];
                y[E + it] = s1[it];
                xs[it] = 0.0, own[it] = 0;
            }
            auto ask = [&](int c) {
                int tk = tid;
                asm volatile("" : "+v"(tk));
#pragma unroll
                for (int it = 0; it < E; it++) {
                    xs[it] = at_lane(special + ((size_t)(c * L) << LOGN) + it * TH, tk);
                    own[it] = at_lane(in + c * comp + it * TH, tk);
                }
            };
            inv_row<LOGN, E, false, sum_bound<2>(), 2>(lds, y, StRegs{y}, 0, tid, itw, m, r, C, 0, [&] { ask(0); });
#pragma unroll
            for (int c = 0; c < 2; c++) {
                int tk = tid;
                asm volatile("" : "+v"(tk));
                double v[E];
#pragma unroll
                for (int it = 0; it < E; it++) v[it] = mulmod(y[c * E + it] - red(xs[it], C->mod[k]), C->Pinv_q[r], m);
                if (c == 0) {
                    lds_barrier();
#pragma unroll
                    for (int it = 0; it < E; it++) lds[tk + it * TH] = u64_to_f64(own[it]);
                    ask(1);     // (component 0's own words are read back from LDS)
                    lds_barrier();
                    int i = 0;
                    do {
                        // terms are canonical up to their sign: four of them between two reductions
                        const uint32_t ginv = H.ginv[i], e0 = (uint32_t)tk * ginv;
#pragma unroll
                        for (int it = 0; it < E; it++) {
                            const uint32_t e = e0 + (uint32_t)(it * TH) * ginv;
                            v[it] = signed_add(v[it], lds[e & (N - 1)], e << (31 - LOGN));
                        }
                        if ((i & 3) == 3) {
#pragma unroll
                            for (int it = 0; it < E; it++) v[it] = red(v[it], m);
                        }
                    } while (++i < H.n_sum);
#pragma unroll
                    for (int it = 0; it < E; it++) v[it] += lds[tk + it * TH];
                } else {
#pragma unroll
                    for (int it = 0; it < E; it++) v[it] += u64_to_f64(own[it]);
                }
#pragma unroll
                for (int it = 0; it < E; it++) put_lane(out + c * comp + it * TH, tk, f64_to_u64(canon(v[it], m)));
            }
        };
        finish(s, s + E, b0);
        if (b0 + 1 < A.batch) {
            lds_barrier();
            finish(s2, s3, b0 + 1);
        }
    }
}

// ---------------------------------------------------------------------------
// The same at N = 16384, for digits of one or two primes: a row is two half rows of 8192 that one workgroup takes through LDS one after the
// other (the first stage, which joins them, in registers; half h is the sub-transform at node 2 + h), and both lie there when the rotations
// take their values, which come from either half.  A relinearisation is the series of one rotation by 1.  What three launches moved through
// memory (a unit's transformed digits out and in, its accumulators out, in and out again: 104 rows of 142 per key switch) never leaves the compute
// unit, and memory is what bounds a step at this size.  Registers: four sums and a half row, as with two units at N = 8192.  Bound by
// vector issue and the keys' way from L2 (5.4 MB a row with 7 rotations).  32 ciphertexts, six primes, two special ones, 7 rotations:
// mod-up, sums and inverse transforms 61 + 101 + 39 us, 135 here, 123 where workgroups begin with different rotations.
// ---------------------------------------------------------------------------
// The constants of a digit's lift to one prime, in scalar registers (as LiftTab)
template <int ALPHA> struct DigitTab {
    ModD ms;
    double inv, s_mod_t;
    __device__ __forceinline__ DigitTab(const DevConst *C, int j, int r) : ms{0.0, 0.0}, inv(0.0), s_mod_t(0.0)
    {
        if constexpr (ALPHA == 2) {
            C = opaque_const(C);
            ms = ModD{pinned(C->mod[2 * j + 1].p), pinned(C->mod[2 * j + 1].u)};
            inv = pinned(C->dig[j].inv[0][1]);
            s_mod_t = pinned(C->dig[j].s_mod_t[0][r]);
        }
    }
    // the digit (an integer in [0, Q_j)) modulo m, below 1.7 * 2^50
    __device__ __forceinline__ double lift(const uint64_t *w, const ModD m) const
    {
        const double x0 = u64_to_f64(w[0]);
        if constexpr (ALPHA == 1) return x0;
        else return mulmod(canon(mulmod(u64_to_f64(w[ALPHA - 1]) - x0, inv, ms), ms), s_mod_t, m) + x0;
    }
};
template <int ALPHA>
__global__ void __launch_bounds__(1024, 4)
ks_wide_kernel(LdModup<false, ALPHA> ld, HoistTab T, int n_rot, int batch, StInvF64 st, const double *__restrict__ tw_all,
               const double *__restrict__ itw_all, const DevConst *__restrict__ C, int nwg)
{
    constexpr int LOGN = 14, E = 8, TH = 1024, HALF = 1 << 13, ROW = lds_doubles<13>();
    constexpr int IN = hundredths(1.7 + 0.5 + 0.1875 * 1.7);
    static_assert(2 * ROW == lds_doubles<14>(), "both halves as one padded row");
    __shared__ __align__(16) double lds[2 * ROW];
    const int tid = threadIdx.x, L = C->L, dnum = C->dnum;
    // as in ks_sum_row_kernel
    const int per_xcd = (nwg + 7) >> 3, total = per_xcd * 8;
    for (int p = blockIdx.x; p < total; p += (int)gridDim.x) {
        const int wg = (p & 7) * per_xcd + (p >> 3);
        if (wg >= nwg) continue;
        const int r = wg / batch, b = wg - r * batch;
        const ModD m = C->mod[r];
        const double *tw = tw_all + ((size_t)r << LOGN), *itw = itw_all + ((size_t)r << LOGN);
        const double w1 = tw[1];
        // half and component
        double s00[E], s01[E], s10[E], s11[E];
#pragma unroll
        for (int it = 0; it < E; it++) s00[it] = s01[it] = s10[it] = s11[it] = 0.0;
        for (int j = 0; j < dnum; j++) {
            const uint64_t *src = ld.src + (size_t)b * ld.unit_stride + ((size_t)(j * ALPHA) << LOGN);
            const DigitTab<ALPHA> tab(C, j, r);
            uint64_t w[2][2][ALPHA];
            auto get = [&](int it) {
#pragma unroll
                for (int h = 0; h < 2; h++)
#pragma unroll
                    for (int a = 0; a < ALPHA; a++) w[it & 1][h][a] = at_lane(src + ((size_t)a << LOGN) + h * HALF + it * TH, tid);
            };
            double x[E];
            get(0);
            lds_barrier();      // the previous digit's (or unit's) LDS reads
#pragma unroll
            for (int it = 0; it < E; it++) {
                if (it + 1 < E) get(it + 1);
                __builtin_amdgcn_sched_barrier(0);
                const double a = tab.lift(w[it & 1][0], m), t = mulmod(tab.lift(w[it & 1][1], m), w1, m);
                x[it] = a + t;
                lds[row_pos<13>(1, pad(tid)) + pad(it * TH)] = a - t;      // where the second half's first pass has it
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int h = 0; h < 2; h++) {
                double *row = lds + h * ROW;
                if (h) {
#pragma unroll
                    for (int it = 0; it < E; it++) x[it] = row[pad(tid) + pad(it * TH)];
                }
                fwd_row<13, E, false, false, 1, IN>(row, x, x, tid, tw, m, Nothing(), 2 + h);
#pragma unroll
                for (int it = 0; it < E; it += 2)
                    pair_at(row, pad(chunk_elem<E>(tid, it))) = make_double2(red(x[it], m), red(x[it + 1], m));
            }
            lds_barrier();
            int tk = tid;
            asm volatile("" : "+v"(tk));
            const int idx0 = chunk_elem<E>(tk, 0);
            const uint32_t e0 = 2u * (__brev((uint32_t)idx0) >> (32 - LOGN)) + 1u;
            const size_t comp = (size_t)L << (LOGN - 1);
            auto rows = [&](int i) { return reinterpret_cast<const cg_double2v *>(T.key[i] + ((size_t)(2 * j * L + r) << LOGN)); };
            // Workgroups begin with different rotations: all at the same one, every key's first trip from memory held all of them up.  Series of 7
            // rotations, 32 ciphertexts 208 -> 195 us, 48: 354 -> 340; 15, 32: 305 -> 286.  (At N = 8192 no difference.)
            int at_rot = b % n_rot;
            const cg_double2v *k0 = rows(at_rot);
            uint32_t g = T.g[at_rot];
            cg_double2v ka[2], kc[2];
            ka[0] = at_lane(k0, idx0 / 2);
            kc[0] = at_lane(k0 + comp, idx0 / 2);
            for (int i = 0; i < n_rot; i++) {
                at_rot = at_rot + 1 < n_rot ? at_rot + 1 : 0;
                const cg_double2v *kn = rows(at_rot);
                const uint32_t gn = T.g[at_rot], eg = __umul24(e0, g);
#pragma unroll
                for (int f = 0; f < E; f++) {       // pair f % 4 of half f / 4, its keys asked for one ahead
                    const cg_double2v *kf = f + 1 < E ? k0 + (f + 1) / 4 * (HALF / 2) + 64 * ((f + 1) % 4) : kn;
                    ka[(f + 1) & 1] = at_lane(kf, idx0 / 2);
                    kc[(f + 1) & 1] = at_lane(kf + comp, idx0 / 2);
                    __builtin_amdgcn_sched_barrier(0);
                    const cg_double2v a = ka[f & 1], c = kc[f & 1];
                    const int q = f % 4;
                    const uint32_t e = eg + (2u * (__brev((uint32_t)(128 * q)) >> (32 - LOGN)) + 2u * (f / 4)) * g;
                    const int at = pad((int)((__brev(e) >> (31 - LOGN)) & ((1u << LOGN) - 1u)));
                    const double x0 = lds[at], x1 = lds[at ^ 1];
                    double (&d0)[E] = f < 4 ? s00 : s10, (&d1)[E] = f < 4 ? s01 : s11;
                    d0[2 * q] += mulmod(x0, a.x, m);
                    d0[2 * q + 1] += mulmod(x1, a.y, m);
                    d1[2 * q] += mulmod(x0, c.x, m);
                    d1[2 * q + 1] += mulmod(x1, c.y, m);
                    __builtin_amdgcn_sched_barrier(0);
                }
                k0 = kn;
                g = gn;
                // a term is below 0.6 p
                if ((i & 7) == 7 || i + 1 == n_rot) {
#pragma unroll
                    for (int it = 0; it < E; it++) {
                        s00[it] = red(s00[it], m);
                        s01[it] = red(s01[it], m);
                        s10[it] = red(s10[it], m);
                        s11[it] = red(s11[it], m);
                    }
                }
            }
        }
        const double n0 = C->ninv[r], n1 = C->itw1_ninv[r];
        auto inverse = [&](const double *lo, const double *hi, int c) {
            double a[E], d[E];
            lds_barrier();
            inv_row<13, E, false, 52>(lds, lo, StHalfRegs{{a}}, 0, tid, itw, m, 0, C, 0, Nothing(), 2);
            inv_row<13, E, false, 52>(lds + ROW, hi, StHalfRegs{{d}}, 0, tid, itw, m, 0, C, 0, Nothing(), 3);
            double *o = st.dst + ((size_t)((b * 2 + c) * L + r) << LOGN);
#pragma unroll
            for (int it = 0; it < E; it++) {
                put_lane(o + it * TH, tid, mulmod(a[it] + d[it], n0, m));
                put_lane(o + HALF + it * TH, tid, mulmod(a[it] - d[it], n1, m));
            }
        };
        inverse(s00, s10, 0);
        inverse(s01, s11, 1);
    }
}

// ---------------------------------------------------------------------------
// Products of ciphertexts, one (unit, prime) per workgroup: transforms of the operands' four polynomials,
// tensor product and the three inverse transforms in one kernel.  An operand that is there in transformed
// form already (an a operand shared by several units, a cache with a transformed copy) is read in it.
// Instead of 101 rows of traffic per product (three launches: ciphertext primes, auxiliary primes, tensor
// product) 33 reach memory.  An operand's two polynomials go through the forward transform together, the first two components of
// the product through the inverse one: two rows of one prime share the factors and every barrier (seven rows, four walks instead of
// seven), and each has the other's arithmetic to cover its trips to LDS.  Both operands' four rows then lie in registers (114 of 128).
// Bound by vector issue (70 to 73 % of the clocks) and what the operands' words and the stores keep it waiting (16 and 6 %, by leaving them out); the
// clock under this load is 2.0 GHz.  768 products at N = 8192, three primes: 308 + 644 + 764 us for the three launches, 1195 us with
// one row at a time, 1180 in pairs, 1100 with the lift's constants read once besides (in walks of one row these gain nothing: the
// constants' scalar registers are spilled).  Measured without gain: the next rows' first words asked for before the last pass, more of a row's
// words on their way (registers spilled), the stores of all three rows at the end.
// ---------------------------------------------------------------------------
// operands that lift_kernel has lifted, a word per element; loads and conversion apart, so that the words of the next row can be on their way
// during a transform
template <int LOGN, int E>
struct LiftedRow {
    static constexpr int T = (1 << LOGN) / E;
    uint64_t w[E];
    __device__ __forceinline__ void fetch(const uint64_t *src, int r, int tid)
    {
#pragma unroll
        for (int i = 0; i < E; i++) w[i] = at_lane(src + ((size_t)r << LOGN) + i * T, tid);
    }
    __device__ __forceinline__ void finish(double *x) const
    {
#pragma unroll
        for (int i = 0; i < E; i++) x[i] = bits_f64(w[i]);
    }
};

// The constants of a lift to one auxiliary prime, read once and kept in scalar registers.  Read where they are used they were
// asked for anew for every element, six trips to the scalar cache one after the other that nothing covered.
template <int K> struct LiftTab {
    double inv[K][K], s_mod_t[K][1];
    ModD ms[K];
    __device__ __forceinline__ LiftTab(const DevConst *C, int j)
    {
        C = opaque_const(C);
#pragma unroll
        for (int b = 0; b < K; b++) {
            ms[b] = ModD{pinned(C->mod[b].p), pinned(C->mod[b].u)};
            s_mod_t[b][0] = b + 1 < K ? pinned(C->q2b.s_mod_t[b][j]) : 0.0;
#pragma unroll
            for (int a = 0; a < b; a++) inv[a][b] = pinned(C->q2b.inv[a][b]);
        }
    }
};
// The polynomial at src modulo the workgroup's prime (of the k + l), in pass-0 ownership.  A row modulo an auxiliary prime: a pair of elements
// is lifted while the next pair's words are on their way.
template <int LOGN, int E, int K>
__device__ __forceinline__ void lift_row(double *x, const uint64_t *src, int r, int tid, const ModD m, const DevConst *C)
{
    constexpr int T = (1 << LOGN) / E;
    if (r < K) {
#pragma unroll
        for (int it = 0; it < E; it++) x[it] = u64_to_f64(at_lane(src + ((size_t)r << LOGN) + it * T, tid));
        return;
    }
    uint64_t w[2][2][K];
    auto get = [&](int it) {
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
            for (int q = 0; q < K; q++) w[(it >> 1) & 1][i][q] = at_lane(src + ((size_t)q << LOGN) + (it + i) * T, tid);
    };
    get(0);
    const LiftTab<K> tab(C, r - K);
#pragma unroll
    for (int it = 0; it < E; it += 2) {
        // (kept apart: the compiler would ask for the whole row first and spill what the caller holds)
        if (it + 2 < E) get(it + 2);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 2; i++) {
            double v[K], dg[K];
#pragma unroll
            for (int q = 0; q < K; q++) v[q] = u64_to_f64(w[(it >> 1) & 1][i][q]);
            garner_balanced<K>(tab, tab.ms, v, dg);
            x[it + i] = horner<K>(tab, m, dg, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// HAT: 0 both operands in coefficients, 1 the first (x) in coefficients and the second (y) transformed.
// K = 0: half rows at N = 16384, lifted ahead by lift_kernel, which shares a coefficient's mixed-radix digits between the
// auxiliary primes (lifted per prime in a transform's loader, the digits of six primes took twice the transform itself).  96
// products, six primes: 165 + 438 + 404 us for the transforms of ciphertext and auxiliary rows and the tensor product's inverse,
// 161 + 501 us for lift_kernel and this.
template <int LOGN, int E, int K, bool HAT>
__global__ void __launch_bounds__((1 << LOGN) / E, (min_waves<LOGN, E>()))
mul_row_kernel(MulRowArgs A, StTens<K == 0> st, const double *__restrict__ tw_all, const double *__restrict__ itw_all,
               const DevConst *__restrict__ C, int nwg)
{
    constexpr int T = (1 << LOGN) / E;
    // half rows: priorities take 96 products from 1238 to 1224 us, 5 from 115.3 to 113.4; whole rows: no difference
    constexpr bool PRIO = K == 0;
    constexpr double ONE = prod_of(fwd_out<LOGN>());        // bound of a product
    const int KL = K ? 2 * K + 1 : A.k;
    __shared__ __align__(16) double lds[2 * lds_doubles<LOGN>()];
    const int tid = threadIdx.x;
    for (int p = blockIdx.x; p < nwg; p += (int)gridDim.x) {
        const int wg = xcd_row(p, nwg, KL), r = wg % KL, u = wg / KL;
        const ModD m = C->mod[K ? r : r >> 1];
        const double *tw = tw_all + ((size_t)r << LOGN), *itw = itw_all + ((size_t)r << LOGN);
        auto load = [&](double *x, const uint64_t *p0, const uint64_t *p1) {
            if constexpr (K == 0) {
#pragma unroll
                for (int it = 0; it < E; it++) {
                    x[it] = bits_f64(at_lane(p0 + ((size_t)r << LOGN) + it * T, tid));
                    x[E + it] = bits_f64(at_lane(p1 + ((size_t)r << LOGN) + it * T, tid));
                }
            } else {
                lift_row<LOGN, E, K>(x, p0, r, tid, m, C);
                lift_row<LOGN, E, K>(x + E, p1, r, tid, m, C);
            }
        };
        double x[2 * E], y[2 * E], e[2 * E], z[E];
        load(x, A.x_poly(u, 0), A.x_poly(u, 1));
        if (p != (int)blockIdx.x) lds_barrier();
        fwd_row<LOGN, E, false, PRIO, 2>(lds, x, x, tid, tw, m);
#pragma unroll
        for (int it = 0; it < 2 * E; it++) x[it] = red(x[it], m);
        if constexpr (HAT) {
            const double *y0 = A.y_hat(u, r, KL), *y1 = y0 + ((size_t)KL << LOGN);
            int tk = tid;
            asm volatile("" : "+v"(tk));
#pragma unroll
            for (int it = 0; it < E; it++) {
                y[it] = at32(y0, chunk_elem<E>(tk, it));
                y[E + it] = at32(y1, chunk_elem<E>(tk, it));
            }
        } else {
            load(y, A.y_poly(u, 0), A.y_poly(u, 1));
            lds_barrier();
            fwd_row<LOGN, E, false, PRIO, 2>(lds, y, y, tid, tw, m);
        }
#pragma unroll
        for (int it = 0; it < E; it++) {
            e[it] = mulmod(x[it], y[it], m);
            e[E + it] = mulmod(x[it], y[E + it], m) + mulmod(x[E + it], y[it], m);
            z[it] = mulmod(x[E + it], y[E + it], m);
        }
        inv_row<LOGN, E, PRIO, hundredths(2.0 * ONE), 2>(lds, e, st, (u * 3) * KL + r, tid, itw, m, 0, C, KL);
        lds_barrier();
        inv_row<LOGN, E, PRIO, hundredths(ONE)>(lds, z, st, (u * 3 + 2) * KL + r, tid, itw, m, 0, C);
    }
}

// The same for mul_sum_row_kernel, W elements' words on their way while one is lifted.  All workgroups of a round walk over the same
// units, and those of a unit share its words in one L2: lift_row, which is done sooner with rows modulo ciphertext primes, lets them
// drift apart (12 groups of 128, N = 8192: 1590 us here, 1650 with lift_row, 1695 with a branch for the ciphertext primes here).
// fetch asks for the first W elements, and can do so before the products of the row before, which have the registers to spare: contexts
// of 12 heads over 128 products, N = 8192, 2282 -> 2267 us, 10: 1902 -> 1892 (W = 5, which fills the registers: 2288); N = 4096,
// four heads over 64 173.5 -> 167.5, 16: 558 -> 547.
template <int LOGN, int E, int K, int W> struct LiftedWindow {
    static constexpr int T = (1 << LOGN) / E;
    uint64_t w[W][K];
    const uint64_t *src;
    __device__ __forceinline__ void get(int it, int r, int tid)
    {
#pragma unroll
        for (int q = 0; q < K; q++) w[it % W][q] = at_lane(src + ((size_t)LdMulExt<K>::source(r, q) << LOGN) + it * T, tid);
    }
    __device__ __forceinline__ void fetch(const uint64_t *poly, int r, int tid)
    {
        src = poly;
#pragma unroll
        for (int it = 0; it < W; it++) get(it, r, tid);
        __builtin_amdgcn_sched_barrier(0);
    }
    __device__ __forceinline__ void finish(double *x, int r, int tid, const ModD m, const DevConst *C)
    {
        C = opaque_const(C);
#pragma unroll
        for (int it = 0; it < E; it++) {
            // (kept apart: the compiler would ask for the whole row first and spill what the caller holds)
            __builtin_amdgcn_sched_barrier(0);
            x[it] = LdMulExt<K>::lift(w[it % W], r, m, C);
            __builtin_amdgcn_sched_barrier(0);
            if (it + W < E) get(it + W, r, tid);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
};

// How sums' units are divided over the workgroups of a prime.  ranges = 0: every group of `group` units in `stride` parts.  Else the units of
// all groups form one row, cut into as many ranges of one length wherever groups end: the piece of group g that lies in range w is its part
// w - first range of the group.  Results of part q of group g are at slot g * stride + q.
struct SumParts {
    int stride, group, units, ranges;
    // the range that unit x lies in (range w starts at w * units / ranges, rounded down)
    __device__ __forceinline__ int range_of(int x) const { return ((x + 1) * ranges - 1) / units; }
    __device__ __forceinline__ int count(int g) const
    {
        return ranges ? range_of((g + 1) * group - 1) - range_of(g * group) + 1 : stride;
    }
};

// Sums of products over the units of a group, one (group, part of it, prime) or (range, prime) per workgroup (SumParts): the operands of a unit
// transformed as in mul_row_kernel, the three components summed over the units, one inverse transform of each sum.  What
// the parts of a group leave is summed by scale_kernel.  It saves the transformed operands' way through memory, and
// its parts spread long groups over the chip.
// Registers set the pace at N = 8192: three sums, a kept row, the row in work and its factors do not fit 128 and spilled 48
// of them, 200 bytes a thread and transform.  There (FAR) two sums stay in registers; the first component's, needed
// once per unit, waits in its own output row, a thread's own 64 bytes of it, from L2.  The words of a polynomial come in through a
// window of a few elements instead of in two halves at once.  Kernel, 12 groups of 128, N = 8192, three primes: 2100 us with everything
// in registers, 1890 with the halves one after the other, 1760 with the first sum in memory too, 1640 with the window (2 to 5
// elements within 3 %), 1561 with N^-1 left to the scaling and the window's first words asked for ahead; the vector unit is 62 % busy.  At N = 4096 registers suffice, and the sum in memory costs 3 % of A V, 12 heads (419 us; 406 in registers).
// With y transformed at N = 16384 three sums beside the row, its factors and y's words spilled 16 registers; with the first one in
// memory none (mul_sum_parts_half has both sides).
template <int LOGN, int E, int K, bool HAT>
__global__ void __launch_bounds__((1 << LOGN) / E, (min_waves<LOGN, E>()))
mul_sum_row_kernel(MulRowArgs A, SumParts S, StTens<K == 0> st, const double *__restrict__ tw_all,
                   const double *__restrict__ itw_all, const DevConst *__restrict__ C, int nwg)
{
    constexpr int T = (1 << LOGN) / E, W = K == 1 ? 8 : K == 2 ? 4 : 3;
    const int KL = K ? 2 * K + 1 : A.k;
    constexpr bool FAR = LOGN > 12;
    __shared__ __align__(16) double lds[lds_doubles<LOGN>()];
    __shared__ double park[HAT ? 1 : 1 << LOGN];
    // prompt context of twelve heads 2303 -> 2284 us; at N = 4096 a step of sixteen heads 175 -> 190 (fwd_pass)
    constexpr bool PRIO = LOGN == 13 && !HAT;
    constexpr bool AHEAD = K != 0 && !HAT;
    const int tid = threadIdx.x;
    for (int p = blockIdx.x; p < nwg; p += (int)gridDim.x) {
        // (a prime's ranges, or the parts of its groups, one after the other)
        const int wg = xcd_row(p, nwg, KL), r = wg % KL, w = wg / KL, g0 = w / S.stride, part = w - g0 * S.stride;
        int u0 = S.ranges ? w * S.units / S.ranges : g0 * S.group + part * S.group / S.stride;
        const int end = S.ranges ? (w + 1) * S.units / S.ranges : g0 * S.group + (part + 1) * S.group / S.stride;
        const ModD m = C->mod[K ? r : r >> 1];
        const double *tw = tw_all + ((size_t)r << LOGN), *itw = itw_all + ((size_t)r << LOGN);
        while (u0 < end) {
            const int u_first = u0, g = u0 / S.group, u_end = end < (g + 1) * S.group ? end : (g + 1) * S.group;
            const int gp = S.ranges ? g * S.stride + w - S.range_of(g * S.group) : w;
            u0 = u_end;
            // the first component's sum: pair q of a thread at far[q * T + tid]
            cg_double2v *far = reinterpret_cast<cg_double2v *>(st.dst + ((size_t)(gp * 3 * KL + r) << LOGN));
            double d0[E], d1[E], d2[E];
#pragma unroll
            for (int it = 0; it < E; it++) d0[it] = d1[it] = d2[it] = 0.0;
            // polynomials of a unit in the order they are transformed: x0, y0, x1, y1 (HAT: x0, x1)
            constexpr int NT = HAT ? 2 : 4;
            auto poly = [&](int u, int t) {
                return HAT ? A.x_poly(u, t) : ((t & 1) ? A.y_poly(u, t >> 1) : A.x_poly(u, t >> 1));
            };
            // the first component's sum before unit u, and put back with a pair of that unit's products (below 2 p)
            auto far_put = [&](const cg_double2v s, double a, double b, int q, int tk) {
                put32(far + q * T, tk, cg_double2v{red(s.x + a, m), red(s.y + b, m)});
            };
            auto far_get = [&](cg_double2v *s0, int u, int tk) {
#pragma unroll
                for (int q = 0; q < E / 2; q++) s0[q] = cg_double2v{0.0, 0.0};
                if (u != u_first) {
#pragma unroll
                    for (int q = 0; q < E / 2; q++) s0[q] = at_lane(far + q * T, tk);
                }
            };
            LiftedRow<LOGN, E> whole;
            LiftedWindow<LOGN, E, K ? K : 1, W> part;
            if constexpr (K == 0) whole.fetch(poly(u_first, 0), r, tid);
            else if constexpr (AHEAD) part.fetch(poly(u_first, 0), r, tid);
            for (int u = u_first; u < u_end; u++) {
                auto row = [&](double *x, int t) {
                    if constexpr (K == 0) {
                        whole.finish(x);
                        whole.fetch(t + 1 < NT ? poly(u, t + 1) : poly(u + 1 < u_end ? u + 1 : u, 0), r, tid);
                    } else {
                        if constexpr (!AHEAD) part.fetch(poly(u, t), r, tid);
                        part.finish(x, r, tid, m, C);
                    }
                };
                if constexpr (HAT) {
                    const double *y0 = A.y_hat(u, r, KL), *y1 = y0 + ((size_t)KL << LOGN);
#pragma unroll
                    for (int t = 0; t < 2; t++) {
                        double x[E];
                        row(x, t);
                        lds_barrier();      // the previous transform's LDS reads
                        fwd_row<LOGN, E, false, PRIO>(lds, x, x, tid, tw, m);
                        int tk = tid;
                        asm volatile("" : "+v"(tk));
                        cg_double2v s0[E / 2];
                        if (FAR && t == 0) far_get(s0, u, tk);
#pragma unroll
                        for (int it = 0; it < E; it++) {
                            const double b0 = at32(y0, chunk_elem<E>(tk, it)), b1 = at32(y1, chunk_elem<E>(tk, it));
                            x[it] = red(x[it], m);
                            if (t == 0) {
                                d1[it] += mulmod(x[it], b1, m);
                                x[it] = mulmod(x[it], b0, m);
                                if (!FAR) d0[it] += x[it];
                                else if (it & 1) far_put(s0[it / 2], x[it - 1], x[it], it / 2, tk);
                            } else {
                                d1[it] += mulmod(x[it], b0, m);
                                d2[it] += mulmod(x[it], b1, m);
                            }
                        }
                    }
                } else {
                    double keep[E];
#pragma unroll
                    for (int t = 0; t < 4; t++) {
                        double x[E];
                        row(x, t);
                        lds_barrier();      // the previous transform's LDS reads
                        fwd_row<LOGN, E, false, PRIO>(lds, x, x, tid, tw, m);
                        cg_double2v s0[E / 2];
                        int tk = tid;
                        asm volatile("" : "+v"(tk));
                        if (FAR && t == 1) far_get(s0, u, tk);
                        if constexpr (AHEAD) part.fetch(t + 1 < NT ? poly(u, t + 1) : poly(u + 1 < u_end ? u + 1 : u, 0), r, tid);
#pragma unroll
                        for (int it = 0; it < E; it++) {
                            if (t % 2 == 0) x[it] = red(x[it], m);      // (one factor of every product)
                            if (t == 0) park[tid + it * T] = x[it];
                            if (!FAR && t == 1) d0[it] += mulmod(park[tid + it * T], x[it], m);
                            if (t == 2) d1[it] += mulmod(x[it], keep[it], m);
                            if (t == 3) {
                                d1[it] += mulmod(park[tid + it * T], x[it], m);
                                d2[it] += mulmod(x[it], keep[it], m);
                            }
                            if (t == 1 || t == 2) keep[it] = x[it];
                        }
                        if (FAR && t == 1) {
#pragma unroll
                            for (int q = 0; q < E / 2; q++)
                                far_put(s0[q], mulmod(park[tid + 2 * q * T], x[2 * q], m),
                                        mulmod(park[tid + (2 * q + 1) * T], x[2 * q + 1], m), q, tk);
                        }
                    }
                }
#pragma unroll
                for (int it = 0; it < E; it++) {
                    if (!FAR) d0[it] = red(d0[it], m);
                    d1[it] = red(d1[it], m);
                    d2[it] = red(d2[it], m);
                }
            }
#pragma unroll
            for (int q = 0; FAR && q < E / 2; q++) {
                const cg_double2v v = at_lane(far + q * T, tid);
                d0[2 * q] = v.x;
                d0[2 * q + 1] = v.y;
            }
            for (int c = 0; c < 3; c++) {
                // (before the first one: the previous transform's LDS reads; every thread has its part of the first sum in
                // registers before any thread stores results over it)
                lds_barrier();
                inv_row<LOGN, E, PRIO, 52>(lds, d0, st, (gp * 3 + c) * KL + r, tid, itw, m, 0, C);
#pragma unroll
                for (int it = 0; it < E; it++) {
                    d0[it] = d1[it];
                    d1[it] = d2[it];
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// ct x pt in one kernel: forward transform of a row, product with the prepared plaintext row, inverse
// transform, the row staying in LDS throughout.  A row crosses memory once in each direction (plus
// the plaintext row, which all ciphertexts of a call share or stream), where the transforms as two
// launches moved it twice and wrote and read the transformed row.
// ---------------------------------------------------------------------------
// storer of the forward half: multiplies in place (a thread's own elements of its wave's chunk)
template <int E, bool PF>
struct StTimesPlain {
    double *lds;
    const double *row;     // plaintext row
    const double *pl;      // PF: its values at the thread's elements, brought in ahead
    __device__ __forceinline__ void store(int it, int idx, double v, const ModD m) const
    {
        lds[pad(idx)] = mulmod(v, PF ? pl[it] : row[idx], m);
    }
};
template <int E, bool PF> struct st_in_place<StTimesPlain<E, PF>> { static constexpr bool value = true; };
template <int LOGN, int E, class ST>
__global__ void __launch_bounds__((1 << LOGN) / E, (min_waves<LOGN, E>()))
ntt_mulplain_kernel(const uint64_t *__restrict__ src, const double *__restrict__ plain, int pstride, int pofs, ST st,
                    const double *__restrict__ tw_all, const double *__restrict__ itw_all,
                    const DevConst *__restrict__ C, int nwg)
{
    __shared__ __align__(16) double lds[lds_doubles<LOGN>()];
    constexpr int T = (1 << LOGN) / E, NP = Plan<LOGN, E>::NP;
    constexpr int IN = hundredths(prod_of(FwdBound<LOGN, E, NP - 1>::out));
    // the plaintext row and the next row are brought in ahead where there are registers for it
    constexpr bool PF = prefetch_rows<LOGN, E>();
    static_assert(NP == 4 || NP == 5, "pass sequence below");
    // 128 appends of 24 ciphertexts, N = 8192: 1981 -> 1928 us; 64 of 24, N = 4096: 524 -> 506; N = 16384: 1895 -> 1976
    constexpr bool PRIO = LOGN <= 13;
    const int tid = threadIdx.x, k = C->k;
    uint64_t raw[E];
    int wg = blockIdx.x;
    auto fetch = [&](int w) {
#pragma unroll
        for (int it = 0; it < E; it++) raw[it] = at_lane(src + ((size_t)w << LOGN) + it * T, tid);
    };
    if constexpr (PF) fetch(wg);
    for (;;) {
        const int pr = wg % k;
        const ModD m = C->mod[pr];
        const auto str = st.at_row(wg, k);
        const double *tw = tw_all + ((size_t)pr << LOGN), *itw = itw_all + ((size_t)pr << LOGN);
        const double *prow = plain + ((size_t)(((wg / (2 * k)) * pstride + pofs) * k + pr) << LOGN);
        double twa[TWREGS], twb[TWREGS], in[E], pl[PF ? E : 1];
        load_tw<LOGN, E, 0, true>(tw, tid, twa);
        if constexpr (PF) {
#pragma unroll
            for (int it = 0; it < E; it += 2) {
                const cg_double2v w = at_lane(reinterpret_cast<const cg_double2v *>(prow) + 32 * it, chunk_elem<E>(tid, 0) / 2);
                pl[it] = w.x;
                pl[it + 1] = w.y;
            }
        } else {
            fetch(wg);
        }
#pragma unroll
        for (int it = 0; it < E; it++) in[it] = u64_to_f64(raw[it]);
        const StTimesPlain<E, PF> times{lds, prow, pl};
        fwd_pass<LOGN, E, 0, true>(lds, in, times, tid, tw, twa, twb, m, 0, PRIO);
        fwd_pass<LOGN, E, 1, false>(lds, in, times, tid, tw, twb, twa, m, 0, PRIO);
        fwd_pass<LOGN, E, 2, false>(lds, in, times, tid, tw, twa, twb, m, 0, PRIO);
        fwd_pass<LOGN, E, 3, false>(lds, in, times, tid, tw, twb, twa, m, 0, PRIO);
        if constexpr (NP > 4) fwd_pass<LOGN, E, 4, false>(lds, in, times, tid, tw, twa, twb, m, 0, PRIO);
        load_tw<LOGN, E, NP - 1, false>(itw, tid, twa);
        wave_sync();
        if constexpr (NP > 4) {
            inv_pass<LOGN, E, 4, IN>(lds, str, wg, tid, itw, twa, twb, m, pr, C, nullptr, nullptr, PRIO);
            inv_pass<LOGN, E, 3, IN>(lds, str, wg, tid, itw, twb, twa, m, pr, C, nullptr, nullptr, PRIO);
        } else {
            inv_pass<LOGN, E, 3, IN>(lds, str, wg, tid, itw, twa, twa, m, pr, C, nullptr, nullptr, PRIO);
        }
        inv_pass<LOGN, E, 2, IN>(lds, str, wg, tid, itw, twa, twb, m, pr, C, nullptr, nullptr, PRIO);
        // What the storer adds to is asked for late: loads return in order, so ahead of the passes' factors it would hold
        // these up (the factors of the last two passes are scalar loads).  24 caches of N = 8192: 2008 us before the
        // last pass but one, 1982 before the last; N = 16384: 2059 and 1892; twelve caches of N = 4096: 526 and 537.
        constexpr bool adds = st_adds<decltype(str)>::value, ahead = LOGN <= 12;
        uint64_t old[8];
        if constexpr (adds && ahead) str.template fetch<T>(old, tid, 0);
        inv_pass<LOGN, E, 1, IN>(lds, str, wg, tid, itw, twb, twa, m, pr, C, nullptr, nullptr, PRIO);
        const int next = wg + (int)gridDim.x;
        if constexpr (PF) {
            if (next < nwg) fetch(next);
        }
        if constexpr (adds && !ahead) str.template fetch<T>(old, tid, 0);
        inv_pass<LOGN, E, 0, IN>(lds, str, wg, tid, itw, twa, twb, m, pr, C, nullptr, old, PRIO);
        if (next >= nwg) break;
        wg = next;
        lds_barrier();   // pass 0's LDS reads precede the next row's LDS writes
    }
}

// ---------------------------------------------------------------------------
// Rows in parts, for launches of few rows: a row of 8192 keeps the four SIMDs of a compute unit busy for 4.6 us while most of the chip
// idles.  2^LS workgroups share a row without exchanging anything: of a forward transform part h computes the outputs whose highest index
// bits are h, of an inverse one those whose lowest bits are h, from the first LS stages taken in registers, which every part does for itself
// (at most three products per element), and a transform of N / 2^LS.  The inverse transform's results land 2^LS words apart.
// One product with relinearisation at N = 8192 48.5 -> 44.9 us, at N = 16384 99.9 -> 89.7, a step of one head 171 -> 152 to 167.
// ---------------------------------------------------------------------------
template <class LD, class ST> struct in_parts { static constexpr bool value = false; };
template <class ST> struct StPart {        // forward: the row's part from `at` on
    ST st;
    int at;
    __device__ __forceinline__ void store(int limb, int idx, double v, const ModD m) const { st.store(limb, at + idx, v, m); }
};
template <int LS, class ST> struct StEvery {        // inverse: every 2^LS-th element from `at` on
    ST st;
    int at;
    __device__ __forceinline__ void store(int wg, int idx, double v, const ModD m) const { st.store(wg, (idx << LS) + at, v, m); }
    __device__ __forceinline__ void store_lane(int wg, int idx, int lane, double v, const ModD m) const
    {
        st.store_lane(wg, (idx << LS) + at, lane << LS, v, m);
    }
};

template <int LOGN, int LS, class LD, class ST>
__global__ void __launch_bounds__(1 << (LOGN - LS - 3))
ntt_fwd_part_kernel(LD ld, ST st, const double *__restrict__ tw_all, const DevConst *__restrict__ C, int nwg)
{
    constexpr int SUB = LOGN - LS, E = 8, T = (1 << SUB) / E, NP = Plan<SUB, E>::NP, PARTS = 1 << LS;
    constexpr int IN = hundredths(fwd_grow(FWD_IN, LS));
    static_assert(LS == 1 || LS == 2, "two or four parts");
    __shared__ __align__(16) double lds[lds_doubles<SUB>()];
    const int tid = threadIdx.x;
    // the parts of a row are neighbours on one XCD
    const int q0 = xcd_row((int)blockIdx.x, nwg << LS, PARTS), wg = q0 >> LS, h = q0 & (PARTS - 1), root = PARTS + h;
    const int pr = ld.prime(wg, C);
    const ModD m = C->mod[pr];
    const double *tw = tw_all + ((size_t)pr << LOGN);
    const int dl = ld.dst_limb(wg, C);
    // factors of the first stages, with the sign of this part's outputs
    const double w0 = (h >> (LS - 1)) ? -tw[1] : tw[1], w1 = LS < 2 ? 0.0 : (h & 1) ? -tw[2 + (h >> 1)] : tw[2 + (h >> 1)];
    double in[E], twa[TWREGS], twb[TWREGS];
    auto first = [&](int it, const double *x) {
        if (LS == 1) in[it] = x[0] + mulmod(x[1], w0, m);
        else in[it] = x[0] + mulmod(x[PARTS / 2], w0, m) + mulmod(x[1] + mulmod(x[PARTS - 1], w0, m), w1, m);
    };
    uint64_t raw[E][PARTS][LD::kRaw];
    static_assert(!LD::kScatter, "elements in the order of their places");
    auto at = [&](int it, int q) { return tid + it * T + (q << SUB); };
#pragma unroll
    for (int it = 0; it < E; it++)
#pragma unroll
        for (int q = 0; q < PARTS; q++) ld.fetch(wg, at(it, q), C, raw[it][q]);
#pragma unroll
    for (int it = 0; it < E; it++) {
        double x[PARTS];
#pragma unroll
        for (int q = 0; q < PARTS; q++) x[q] = ld.finish(raw[it][q], wg, at(it, q), m, C);
        first(it, x);
    }
    const StPart<ST> part{st, h << SUB};
    load_tw<SUB, E, 0, true>(tw, tid, twa, root);
    fwd_pass<SUB, E, 0, true, 1, IN>(lds, in, part, tid, tw, twa, twb, m, dl, false, root);
    fwd_pass<SUB, E, 1, false, 1, IN>(lds, in, part, tid, tw, twb, twa, m, dl, false, root);
    fwd_pass<SUB, E, 2, false, 1, IN>(lds, in, part, tid, tw, twa, twb, m, dl, false, root);
    fwd_pass<SUB, E, 3, false, 1, IN>(lds, in, part, tid, tw, twb, twa, m, dl, false, root);
    if constexpr (NP > 4) fwd_pass<SUB, E, 4, false, 1, IN>(lds, in, part, tid, tw, twa, twb, m, dl, false, root);
}

template <int LOGN, int LS, class LD, class ST>
__global__ void __launch_bounds__(1 << (LOGN - LS - 3))
ntt_inv_part_kernel(LD ld, ST st, const double *__restrict__ itw_all, const DevConst *__restrict__ C, int nwg)
{
    constexpr int SUB = LOGN - LS, E = 8, NP = Plan<SUB, E>::NP, PARTS = 1 << LS, N = 1 << LOGN;
    constexpr int IN = hundredths(0.51 * PARTS);       // (a product of sums is smaller)
    static_assert(LS == 1 || LS == 2, "two or four parts");
    __shared__ __align__(16) double lds[lds_doubles<SUB>()];
    const int tid = threadIdx.x;
    const int q0 = xcd_row((int)blockIdx.x, nwg << LS, PARTS), wg = q0 >> LS, h = q0 & (PARTS - 1);
    const int pr = ld.prime(wg, C), orow = __builtin_amdgcn_readfirstlane(ld.out_row(wg, C));
    const ModD m = C->mod[pr];
    const double *itw = itw_all + ((size_t)pr << LOGN);
    const bool low = h & 1, high = LS > 1 && (h & 2);
    double twa[TWREGS], twb[TWREGS];
    load_tw<SUB, E, NP - 1, false>(itw, tid, twa);
    // the first stages' factors, asked for before anything waits
    double f[E][3];
#pragma unroll
    for (int it = 0; it < E; it++) {
        const int j = chunk_elem<E>(tid, it);
        f[it][0] = at32(itw + N / 2, (PARTS / 2) * j);
        f[it][1] = LS > 1 ? at32(itw + N / 2 + 1, 2 * j) : 0.0;
        f[it][2] = LS > 1 ? at32(itw + N / 4, j) : 0.0;
    }
    auto first = [&](int it, const double *x) {
        double a = low ? mulmod(x[0] - x[1], f[it][0], m) : x[0] + x[1];
        if (LS == 1) return a;
        double b = low ? mulmod(x[PARTS - 2] - x[PARTS - 1], f[it][1], m) : x[PARTS - 2] + x[PARTS - 1];
        return high ? mulmod(a - b, f[it][2], m) : a + b;
    };
    uint64_t raw[E][PARTS][LD::kRaw];
#pragma unroll
    for (int it = 0; it < E; it++)
#pragma unroll
        for (int q = 0; q < PARTS; q++) ld.fetch(wg, (chunk_elem<E>(tid, it) << LS) + q, C, raw[it][q]);
    double y[E];
#pragma unroll
    for (int it = 0; it < E; it++) {
        double x[PARTS];
#pragma unroll
        for (int q = 0; q < PARTS; q++) x[q] = red(ld.finish(raw[it][q], wg, (chunk_elem<E>(tid, it) << LS) + q, m, C), m);
        y[it] = first(it, x);
    }
#pragma unroll
    for (int it = 0; it < E; it += 2) pair_at(lds, pad(chunk_elem<E>(tid, it))) = make_double2(y[it], y[it + 1]);
    wave_sync();
    const StEvery<LS, ST> every{st, h};
    static_assert(NP == 4, "parts of 4096");
    inv_pass<SUB, E, 3, IN>(lds, every, orow, tid, itw, twa, twb, m, pr, C);
    inv_pass<SUB, E, 2, IN>(lds, every, orow, tid, itw, twb, twa, m, pr, C);
    inv_pass<SUB, E, 1, IN>(lds, every, orow, tid, itw, twa, twb, m, pr, C);
    inv_pass<SUB, E, 0, IN>(lds, every, orow, tid, itw, twb, twa, m, pr, C);
}
// Loaders that bring in a word or two per element.  Those that work for an element (lifts, tensor and inner products) would do so 2^LS
// times: one product at N = 8192, four parts, operands 13.7 -> 13.1 us, tensor product 12.6 -> 15.3, inner product 11.1 -> 12.9.
template <> struct in_parts<LdRowsU64, StU64> { static constexpr bool value = true; };
// (not mod-ups with a map: chains of rotations of 4 x 4 ciphertexts, N = 8192, 353 us a step with whole rows, 371 in parts; 4 x 1, N = 16384,
// 653 / 738)
template <int A> struct in_parts<LdModup<false, A>, StU64> { static constexpr bool value = true; };
template <> struct in_parts<LdInvU64, StInvU64> { static constexpr bool value = true; };
template <> struct in_parts<LdInvF64, StInvF64> { static constexpr bool value = true; };

// ---------------------------------------------------------------------------
// pointwise kernels
// ---------------------------------------------------------------------------
constexpr int PW_THREADS = 256;

// exact round(t e / Q) mod Q from e known modulo Q and the auxiliary basis:
//   r = centred (t e mod Q);  y = (t e - r) / Q computed modulo each b_j;
//   y is below B/2 in magnitude, so its centred lift from the auxiliary basis is exact.
// tens[(b*parts+q)*3+c][r][n], summed over q (lazy, coefficient order, without the inverse transforms' N^-1) -> out[b][c][i][n] canonical uint64;
// acc != 0 adds the result to what out already holds (sum of products).
// HALF: rows of two half rows whose last inverse stage is still to be taken: the workgroup's waves 0 and 1 take 128
// coefficients of the first half, waves 2 and 3 those of the second that they pair with, and read the same lines.
// 96 products, six primes: 199 us (175 from whole rows, 213 with one thread for both of a pair).
template <int K, bool HALF>
__global__ void __launch_bounds__(PW_THREADS)
scale_kernel(const double *__restrict__ tens, uint64_t *__restrict__ out, SumParts S, int acc,
             const DevConst *__restrict__ C)
{
    constexpr int L = K + 1;
    const int logn = C->logn, chunks = (1 << logn) / PW_THREADS, tid = (int)threadIdx.x;
    const int bc = (int)blockIdx.x / chunks, chunk = (int)blockIdx.x % chunks;
    const int n = HALF ? chunk * (PW_THREADS / 2) + (tid & (PW_THREADS / 2 - 1)) : chunk * PW_THREADS + tid;
    const bool upper = HALF && __builtin_amdgcn_readfirstlane(tid) >= PW_THREADS / 2;
    const size_t half = HALF ? (size_t)1 << (logn - 1) : 0;
    const double *src = tens + (((size_t)((bc / 3) * S.stride * 3 + bc % 3) * (K + L)) << logn);
    const int parts = S.count(bc / 3);
    double e[K + L];
    // element n; HALF: the pair's sum or difference
    auto at = [&](int i) {
        const double *row = src + ((size_t)i << logn);
        if (!HALF) return at32(row, n);
        const double b = at32(row + half, n);
        return at32(row, n) + (upper ? -b : b);
    };
#pragma unroll
    for (int i = 0; i < K + L; i++) e[i] = at(i);
    for (int q = 1; q < parts; q++) {
        src += (size_t)(3 * (K + L)) << logn;
#pragma unroll
        for (int i = 0; i < K + L; i++) e[i] = red(e[i], C->mod[i]) + at(i);
    }
    if (upper) {
#pragma unroll
        for (int i = 0; i < K + L; i++) e[i] = mulmod(e[i], C->itw1[i], C->mod[i]);
    }
    double x[K], dq[K], y[L], db[L];
#pragma unroll
    for (int i = 0; i < K; i++) x[i] = mulmod(e[i], C->t_ninv[i], C->mod[i]);
    garner_balanced<K>(C->q2b, C->mod, x, dq);
#pragma unroll
    for (int j = 0; j < L; j++) {
        const ModD mb = C->mod[K + j];
        const double te = mulmod(e[K + j], C->t_ninv[K + j], mb);
        const double rj = horner<K>(C->q2b, mb, dq, j);
        y[j] = mulmod(te - rj, C->Qinv_b[j], mb);
    }
    garner_balanced<L>(C->b2q, C->mod + K, y, db);
    uint64_t *o = out + (((size_t)bc * K) << logn) + (upper ? half : 0) + n;
#pragma unroll
    for (int i = 0; i < K; i++) {
        double v = canon(horner<L>(C->b2q, C->mod[i], db, i), C->mod[i]);
        if (acc) v = addmod_canon(v, u64_to_f64(o[(size_t)i << logn]), C->mod[i]);
        o[(size_t)i << logn] = f64_to_u64(v);
    }
}

// Operands of products at N = 16384: every polynomial named by src -> its residues modulo the k ciphertext primes and (centred
// lift) the l auxiliary ones, first transform stage taken: rows dst[poly][k+l][2][N/2] of two half rows each, |x| <= FWD_IN 2^50.
// One thread has coefficients n and n + N/2 and shares their mixed-radix digits between the auxiliary primes.
template <int K>
__global__ void __launch_bounds__(PW_THREADS)
lift_kernel(MulSrc src, double *__restrict__ dst, const DevConst *__restrict__ C)
{
    constexpr int L = K + 1;
    const int logn = C->logn, half = 1 << (logn - 1), chunks = half / PW_THREADS;
    const int pp = (int)blockIdx.x / chunks, n = ((int)blockIdx.x % chunks) * PW_THREADS + (int)threadIdx.x;
    const uint64_t *row = src.poly(pp, K);
    double *o = dst + (((size_t)src.dst_poly(pp) * (K + L)) << logn);
    double x[2][K], dg[2][K];
#pragma unroll
    for (int h = 0; h < 2; h++)
#pragma unroll
        for (int i = 0; i < K; i++) x[h][i] = u64_to_f64(at32(row + ((size_t)i << logn) + h * half, n));
    garner_balanced<K>(C->q2b, C->mod, x[0], dg[0]);
    garner_balanced<K>(C->q2b, C->mod, x[1], dg[1]);
#pragma unroll
    for (int r = 0; r < K + L; r++) {
        const ModD m = C->mod[r];
        double a, b;
        if (r < K) {
            a = x[0][r < K ? r : 0];
            b = x[1][r < K ? r : 0];
        } else {
            a = horner<K>(C->q2b, m, dg[0], r - K);
            b = horner<K>(C->q2b, m, dg[1], r - K);
        }
        // |a| <= 0.51, |b w| <= 0.5 + 0.1875 * 1.25: together below 1.25
        a = red(a, m);
        const double t = mulmod(b, C->tw1[r], m);
        put32(o + ((size_t)r << logn), n, a + t);
        put32(o + ((size_t)r << logn) + half, n, a - t);
    }
}

template <bool HOIST, int NSP>
__global__ void __launch_bounds__(PW_THREADS)
moddown_kernel(ModdownArgs A, ModdownHoist H, const DevConst *__restrict__ C)
{
    // a thread takes two neighbouring coefficients: 16 bytes per row and lane on every read and
    // write that is not a permuted one
    const int logn = C->logn, N = 1 << logn, k = C->k, L = C->L;
    // the N / (2 PW_THREADS) blocks of one (unit, component) run on one XCD: the permuted reads of a
    // c0 row touch all of its cache lines, which that XCD's L2 then fetches once instead of once
    // per XCD
    const size_t gid =
        ((size_t)xcd_row((int)blockIdx.x, (int)gridDim.x, N / (2 * PW_THREADS)) * PW_THREADS + threadIdx.x) * 2;
    const int n = (int)(gid & (N - 1));
    const int bc = (int)(gid >> logn);
    if (bc >= A.batch * 2) return;
    const int c = bc & 1;
    int b = bc >> 1, bo = b;       // addend index, output index
    if (HOIST) {
        const int i = b / H.rot_batch;
        b -= i * H.rot_batch;
        bo = b * H.out_per_b + i;
        A.galois = H.ginv[i];
    }
    const double *src = A.acc + (((size_t)bc * L) << logn) + n;
    double xp[2][NSP], dg[2][NSP];
#pragma unroll
    for (int s = 0; s < NSP; s++) {
        const double2 x2 = *reinterpret_cast<const double2 *>(src + ((size_t)(k + s) << logn));
        xp[0][s] = x2.x;
        xp[1][s] = x2.y;
    }
    garner_balanced<NSP>(C->p2q, C->mod + k, xp[0], dg[0]);
    garner_balanced<NSP>(C->p2q, C->mod + k, xp[1], dg[1]);
    int src_idx[2] = {0, 0};
    bool negate[2] = {false, false};
    if (A.galois) {
        // inverse map: output index n takes the coefficient from index n * g^-1 mod 2N
        // (A.galois already holds g^-1 mod 2N)
#pragma unroll
        for (int e2 = 0; e2 < 2; e2++) {
            const uint32_t e = ((uint32_t)(n + e2) * A.galois) & (2 * N - 1);
            negate[e2] = e >= (uint32_t)N;
            src_idx[e2] = (int)(negate[e2] ? e - N : e);
        }
    }
    uint64_t *o = A.out + (size_t)bo * A.out_stride + (((size_t)c * k) << logn) + n;
#pragma unroll
    for (int i = 0; i < MAXS; i++)
        if (i < k) {
            const ModD mq = C->mod[i];
            const double2 a2 = *reinterpret_cast<const double2 *>(src + ((size_t)i << logn));
            const double ain[2] = {a2.x, a2.y};
            double v[2];
#pragma unroll
            for (int e2 = 0; e2 < 2; e2++) {
                v[e2] = mulmod(ain[e2] - horner<NSP>(C->p2q, mq, dg[e2], i), C->Pinv_q[i], mq);
            }
            // addends are canonical: with both the value stays below 2^52 until the one reduction at the end
            if (A.add) {
                const uint64_t *ad = A.add + (size_t)b * A.add_stride;
                if (A.galois) {
                    if (c == 0) {
#pragma unroll
                        for (int e2 = 0; e2 < 2; e2++) {
                            const double w = u64_to_f64(ad[((size_t)i << logn) + src_idx[e2]]);
                            v[e2] += negate[e2] ? -w : w;
                        }
                    }
                    if (A.accumulate) {
                        const uint64_t *aa = A.acc_add + (size_t)b * A.acc_stride;
                        const ulonglong2 w2 =
                            *reinterpret_cast<const ulonglong2 *>(aa + ((size_t)(c * k + i) << logn) + n);
                        v[0] += u64_to_f64(w2.x);
                        v[1] += u64_to_f64(w2.y);
                    }
                } else {
                    const ulonglong2 w2 = *reinterpret_cast<const ulonglong2 *>(ad + ((size_t)(c * k + i) << logn) + n);
                    v[0] += u64_to_f64(w2.x);
                    v[1] += u64_to_f64(w2.y);
                }
            }
            *reinterpret_cast<ulonglong2 *>(o + ((size_t)i << logn)) =
                make_ulonglong2(f64_to_u64(canon(v[0], mq)), f64_to_u64(canon(v[1], mq)));
        }
}

// Mod-down of a summed series of rotations (acc holds the summed accumulators of the H.n_sum
// rotations of ciphertext b), one output row per workgroup: block -> (ciphertext b, component c,
// ciphertext prime i), the prime running fastest.
//   out[b][c][i] = in[b][c][i] + u_{c,i} + [c = 0] sum_r sigma_r(c0)_i
// The Galois maps read c0 at the indices n g_r^-1 mod 2N, a different cache line for every lane;
// the workgroup brings its input row into LDS with coalesced loads and takes the permuted
// coefficients (and the un-permuted addend) from there.  Base conversion as in moddown_kernel,
// for the one prime of the row; the special-prime rows are read by the k workgroups of a
// (ciphertext, component), neighbours on one XCD.
template <int LOGN, int NSP>
__global__ void __launch_bounds__(1024, (LOGN <= 13 ? 8 : 4))
moddown_sum_kernel(ModdownArgs A, ModdownHoist H, const DevConst *__restrict__ C)
{
    // a row is shared by SPLIT workgroups: each parks the whole input row in LDS and produces
    // N / SPLIT of the outputs (SPLIT x k workgroups per ciphertext and component)
    constexpr int N = 1 << LOGN, SPLIT = moddown_sum_split<LOGN>(), ROWP = N / 2048, PAIRS = ROWP / SPLIT;
    static_assert(PAIRS >= 1, "at least one pair of outputs per thread");
    __shared__ double row[N];
    const int k = C->k, L = C->L, tid = threadIdx.x;
    const int blk = xcd_row((int)blockIdx.x, (int)gridDim.x, k * SPLIT);
    const int part = blk % SPLIT, i = (blk / SPLIT) % k, bc = blk / (SPLIT * k), c = bc & 1, b = bc >> 1;
    const ModD mq = C->mod[i];
    const uint64_t *in = A.add + (size_t)b * A.add_stride + ((size_t)(c * k + i) << LOGN);   // row i of c_c
    const double *acc = A.acc + (((size_t)bc * L) << LOGN);
    uint64_t *o = A.out + (size_t)b * A.out_stride + ((size_t)(c * k + i) << LOGN);
    // the input row (component 1: only the part this workgroup produces), and the accumulator
    // operands of the thread's first pairs, are requested before anything waits
    auto pair_index = [&](int j) { return 2 * (tid + 1024 * (part * PAIRS + j)); };
    if (c == 0) {
        ulonglong2 all[ROWP];
#pragma unroll
        for (int j = 0; j < ROWP; j++) all[j] = *reinterpret_cast<const ulonglong2 *>(in + 2 * (tid + 1024 * j));
#pragma unroll
        for (int j = 0; j < ROWP; j++)
            *reinterpret_cast<double2 *>(row + 2 * (tid + 1024 * j)) =
                make_double2(u64_to_f64(all[j].x), u64_to_f64(all[j].y));
    } else {
#pragma unroll
        for (int j = 0; j < PAIRS; j++) {
            const ulonglong2 w = *reinterpret_cast<const ulonglong2 *>(in + pair_index(j));
            *reinterpret_cast<double2 *>(row + pair_index(j)) = make_double2(u64_to_f64(w.x), u64_to_f64(w.y));
        }
    }
    constexpr int PB = PAIRS < 2 ? PAIRS : 2;
    double2 xs[PB][NSP], as[PB];
    auto request = [&](int j0) {
#pragma unroll
        for (int j = 0; j < PB; j++) {
            const int n = pair_index(j0 + j);
#pragma unroll
            for (int s = 0; s < NSP; s++) xs[j][s] = *reinterpret_cast<const double2 *>(acc + ((size_t)(k + s) << LOGN) + n);
            as[j] = *reinterpret_cast<const double2 *>(acc + ((size_t)i << LOGN) + n);
        }
    };
    request(0);
    if (c == 0) __syncthreads();     // component 1 reads back only its own elements
#pragma unroll
    for (int j0 = 0; j0 < PAIRS; j0 += PB) {
        double v[PB][2];
#pragma unroll
        for (int j = 0; j < PB; j++) {
            double xp[2][NSP], dg[2][NSP];
#pragma unroll
            for (int s = 0; s < NSP; s++) {
                xp[0][s] = xs[j][s].x;
                xp[1][s] = xs[j][s].y;
            }
            garner_balanced<NSP>(C->p2q, C->mod + k, xp[0], dg[0]);
            garner_balanced<NSP>(C->p2q, C->mod + k, xp[1], dg[1]);
            const double ain[2] = {as[j].x, as[j].y};
#pragma unroll
            for (int e2 = 0; e2 < 2; e2++)
                v[j][e2] = mulmod(ain[e2] - horner<NSP>(C->p2q, mq, dg[e2], i), C->Pinv_q[i], mq);
        }
        if (j0 + PB < PAIRS) request(j0 + PB);     // the next pairs' operands travel during the LDS reads
#pragma unroll
        for (int j = 0; j < PB; j++) {
            const int n = pair_index(j0 + j);
            if (c == 0)
                for (int r = 0; r < H.n_sum; r++) {
                    // terms are canonical up to their sign: four of them between two reductions
                    uint32_t e = (uint32_t)n * H.ginv[r];
                    v[j][0] = signed_add(v[j][0], row[e & (N - 1)], e << (31 - LOGN));
                    e += H.ginv[r];
                    v[j][1] = signed_add(v[j][1], row[e & (N - 1)], e << (31 - LOGN));
                    if ((r & 3) == 3) {
                        v[j][0] = red(v[j][0], mq);
                        v[j][1] = red(v[j][1], mq);
                    }
                }
            const double2 own = *reinterpret_cast<const double2 *>(row + n);
            *reinterpret_cast<ulonglong2 *>(o + n) =
                make_ulonglong2(f64_to_u64(canon(v[j][0] + own.x, mq)), f64_to_u64(canon(v[j][1] + own.y, mq)));
        }
    }
}

// ---------------------------------------------------------------------------
// One component of one rotation of a hoisted series per workgroup, from the transformed digits to the finished
// ciphertext rows: inner products and inverse transform modulo the special prime, then modulo every ciphertext
// prime, the division by P following in registers.  The permuted c0 row goes through LDS.  The accumulators (8 rows
// written and read per rotation at four primes) never reach memory.  A serial chain of k + 1 transforms, so it needs half
// the chip to be busy to pay off.  N = 8192, 127 rotations, mod-down included: 12 ciphertexts 1164 us in two launches, 675 here, one 118 / 69, with
// digits gathered where they are multiplied, which nothing covered (one workgroup to a unit, 14 us a row, the vector unit
// 51 % busy).  Digits side by side through LDS and words asked for ahead: 657 and 63.6, four 247 -> 225; products added up unreduced besides (DotSum):
// 633, 62.7, 217.  (Words asked for before the whole transform, whose factors then wait behind them: 834; the special prime's residues in memory, which
// leaves registers for 16 elements on 512 threads, two workgroups to a unit: 698.  One digit: 68.5 gathered, 74 through LDS.)
// ---------------------------------------------------------------------------
template <int LOGN, int E, int DNUM>
__global__ void __launch_bounds__((1 << LOGN) / E, (min_waves<LOGN, E>()))
rot_row_kernel(const uint64_t *__restrict__ dig, HoistTab T, ModdownArgs A, ModdownHoist H,
               const double *__restrict__ itw_all, const DevConst *__restrict__ C, int nwg)
{
    __shared__ __align__(16) double lds[lds_doubles<LOGN>()];
    constexpr int TH = (1 << LOGN) / E, N = 1 << LOGN;
    const int tid = threadIdx.x, L = C->L, k = C->k, batch = H.rot_batch;
    for (int p = blockIdx.x; p < nwg; p += (int)gridDim.x) {
        // a rotation's component for all ciphertexts on one XCD: the key rows come into one L2 and the digits stay in all
        const int wg = xcd_row(p, nwg, batch), ic = wg / batch, b = wg - ic * batch, c = ic & 1, i = ic >> 1;
        const uint32_t g = T.g[i], ginv = H.ginv[i];
        const uint64_t *in = A.add + (size_t)b * A.add_stride;
        uint64_t *out = A.out + (size_t)(b * H.out_per_b + i) * A.out_stride + ((size_t)(c * k) << LOGN);
        // The map takes every aligned block of 2^m values to such a block: a pair of elements of a wave's lanes reads 128 neighbours.  With several digits these
        // come in side by side, as the keys do, and are permuted in the wave's own part of LDS.
        constexpr bool AHEAD = DNUM > 1;
        const int idx0 = chunk_elem<E>(tid, 0);
        const uint32_t eg = __umul24(2u * (__brev((uint32_t)idx0) >> (32 - LOGN)) + 1u, g);
        uint32_t at[E / 4];     // two to a register: with them apart the kernel for three digits spilled two
        int from[E / 2];
#pragma unroll
        for (int q = 0; q < E / 2; q++) {
            const uint32_t e = eg + 2u * (__brev((uint32_t)(128 * q)) >> (32 - LOGN)) * g;
            const int full = (int)((__brev(e) >> (31 - LOGN)) & (N - 1u));      // as in sum_pairs
            const uint32_t to = (uint32_t)pad((idx0 & ~127) + 128 * q + (full & 127));
            at[q / 2] = q % 2 ? at[q / 2] | to << 16 : to;
            from[q] = __builtin_amdgcn_readfirstlane(full) & ~127;
        }
        cg_ulong2v dv[E / 2];
        cg_double2v kv[E / 2];
        auto ask_digit = [&](int r, int j, int tk) {
            const cg_ulong2v *d = reinterpret_cast<const cg_ulong2v *>(dig + (((size_t)(b * DNUM + j) * L + r) << LOGN));
#pragma unroll
            for (int q = 0; q < E / 2; q++) dv[q] = at_lane(d + from[q] / 2, tk & 63);
        };
        auto ask_key = [&](int r, int j, int tk) {
            const cg_double2v *kb = reinterpret_cast<const cg_double2v *>(T.key[i] + (((size_t)(2 * j + c) * L + r) << LOGN));
#pragma unroll
            for (int q = 0; q < E / 2; q++) kv[q] = at_lane(kb + 64 * q, chunk_elem<E>(tk, 0) / 2);
        };
        if (AHEAD) {
            ask_digit(k, 0, tid);
            ask_key(k, 0, tid);
        }
        double xs[E];
        for (int step = 0; step < L; step++) {
            const int r = step ? step - 1 : k, r_next = step + 1 < L ? step : r;
            const ModD m = C->mod[r];
            const double *itw = itw_all + ((size_t)r << LOGN);
            double y[E];
            int tk = tid;
            asm volatile("" : "+v"(tk));
            if constexpr (AHEAD) {
                static_assert(DNUM <= DotSum::CANONICAL, "canonical digits times centred keys, one sum for all digits");
                DotSum sum[E];
#pragma unroll
                for (int it = 0; it < E; it++) sum[it].open(0.0);
                lds_barrier();      // the previous reads of this wave's part
                // a digit's words are asked for as soon as the last one's have left their registers
#pragma unroll
                for (int j = 0; j < DNUM; j++) {
#pragma unroll
                    for (int q = 0; q < E / 2; q++)
                        pair_at(lds, pad(chunk_elem<E>(tk, 0)) + pad(128 * q)) = make_double2(u64_to_f64(dv[q].x), u64_to_f64(dv[q].y));
                    if (j + 1 < DNUM) ask_digit(r, j + 1, tk);
                    wave_sync();
#pragma unroll
                    for (int q = 0; q < E / 2; q++) {
                        const uint32_t to = q % 2 ? at[q / 2] >> 16 : at[q / 2] & 0xFFFFu;
                        sum[2 * q].add(lds[to], kv[q].x);
                        sum[2 * q + 1].add(lds[to ^ 1], kv[q].y);
                    }
                    if (j + 1 < DNUM) ask_key(r, j + 1, tk);
                    wave_sync();
                }
#pragma unroll
                for (int it = 0; it < E; it++) y[it] = sum[it].close(m);
            } else {
                const cg_ulong2v *d = reinterpret_cast<const cg_ulong2v *>(dig + (((size_t)b * L + r) << LOGN));
                const cg_double2v *kb = reinterpret_cast<const cg_double2v *>(T.key[i] + (((size_t)c * L + r) << LOGN));
                const int idx = chunk_elem<E>(tk, 0);
                const uint32_t ek = __umul24(2u * (__brev((uint32_t)idx) >> (32 - LOGN)) + 1u, g);
#pragma unroll
                for (int q = 0; q < E / 2; q++) {
                    const uint32_t e = ek + 2u * (__brev((uint32_t)(128 * q)) >> (32 - LOGN)) * g;
                    const int full = (int)((__brev(e) >> (31 - LOGN)) & (N - 1u));
                    const cg_double2v kq = at_lane(kb + 64 * q, idx / 2);
                    const cg_ulong2v dq = at32(d, full >> 1);
                    y[2 * q] = mulmod(u64_to_f64((full & 1) ? dq.y : dq.x), kq.x, m);
                    y[2 * q + 1] = mulmod(u64_to_f64((full & 1) ? dq.x : dq.y), kq.y, m);
                }
                lds_barrier();
            }
            // the next prime's first words travel during the last two passes and the division
            inv_row<LOGN, E, false, AHEAD ? hundredths(DotSum::OUT) : 70>(lds, y, StRegs{y}, 0, tid, itw, m, r, C, 0, [&] {
                if (!AHEAD) return;
                int ta = tid;
                asm volatile("" : "+v"(ta));
                ask_digit(r_next, 0, ta);
                ask_key(r_next, 0, ta);
            });
            asm volatile("" : "+v"(tk));
            if (!step) {
#pragma unroll
                for (int it = 0; it < E; it++) xs[it] = red(y[it], m);     // centred residue modulo the special prime
                continue;
            }
#pragma unroll
            for (int it = 0; it < E; it++) y[it] = mulmod(y[it] - xs[it], C->Pinv_q[r], m);
            if (c == 0) {
                uint64_t own[E];
#pragma unroll
                for (int it = 0; it < E; it++) own[it] = at_lane(in + ((size_t)r << LOGN) + it * TH, tk);
                lds_barrier();
#pragma unroll
                for (int it = 0; it < E; it++) lds[tk + it * TH] = u64_to_f64(own[it]);
                lds_barrier();
#pragma unroll
                for (int it = 0; it < E; it++) {
                    const uint32_t e = (uint32_t)(tk + it * TH) * ginv;
                    y[it] = signed_add(y[it], lds[e & (N - 1)], e << (31 - LOGN));
                }
            }
#pragma unroll
            for (int it = 0; it < E; it++)
                put32(out + ((size_t)r << LOGN) + it * TH, tk, f64_to_u64(canon(y[it], m)));
        }
    }
}

// A digit's transformed values times its two key rows, added to two sums.  Keys are asked for a pair of elements ahead, the first
// one before the transform's last pass: all of them asked for after the transform, every wave waited there for the
// 128 KB that a compute unit takes in at 39 bytes a clock.  768 products and relinearisations at N = 8192 1925 -> 1877 us,
// at N = 4096 572 -> 562.  (The next digit's words asked for as late as that: 1901.  In ks_row_kernel
// and for rotations it gains nothing: the step's launches of 48 units are 0.6 % slower.)
template <int LOGN, int E>
struct DigitKeys {
    const cg_double2v *k0, *k1;
    int lane;
    cg_double2v a[2], c[2];
    __device__ __forceinline__ DigitKeys(const double *key, size_t comp, int tid)
        : k0(reinterpret_cast<const cg_double2v *>(key)), k1(reinterpret_cast<const cg_double2v *>(key + comp)),
          lane(chunk_elem<E>(tid, 0) / 2) {}
    __device__ __forceinline__ void ask(int q)
    {
        a[q & 1] = at32(k0, lane + 64 * q);
        c[q & 1] = at32(k1, lane + 64 * q);
    }
    __device__ __forceinline__ void add(const double *x, const ModD m, double *s0, double *s1)
    {
#pragma unroll
        for (int q = 0; q < E / 2; q++) {
            if (q + 1 < E / 2) ask(q + 1);
            __builtin_amdgcn_sched_barrier(0);
            const cg_double2v ka = a[q & 1], kc = c[q & 1];
            s0[2 * q] += mulmod(x[2 * q], ka.x, m);
            s0[2 * q + 1] += mulmod(x[2 * q + 1], ka.y, m);
            s1[2 * q] += mulmod(x[2 * q], kc.x, m);
            s1[2 * q + 1] += mulmod(x[2 * q + 1], kc.y, m);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
};

// ---------------------------------------------------------------------------
// Key switch of one unit per workgroup, from the ring element to the finished ciphertext: as ks_row_kernel and
// ks_sum_row_kernel, special prime first, then every ciphertext prime with the division by P and the additions in
// registers.  The accumulators (L rows of each component written and read again) never reach memory but for the two
// rows modulo the special prime, and the mod-down launch is gone.  The vector unit is 53 to 56 % busy in rotations and 63 to 66 % in
// relinearisations, less than in those kernels: the addends, asked for before the last two passes of the inverse transforms
// (after them, and with one sum at a time: 768 relinearisations 522 us against 495), are in part exposed.  us by row / by unit, N = 8192, 768 units: relinearisation 553 / 459, rotation
// 580 / 537, 3 summed rotations 700 / 698; N = 4096: 154 / 128, 158 / 144, 7 summed 259 / 215.
// ---------------------------------------------------------------------------
enum KsMode { KS_PLAIN, KS_ROTATE, KS_SUM };
template <int LOGN, int E, int MODE>
__global__ void __launch_bounds__((1 << LOGN) / E, (MODE == KS_ROTATE ? 4 : min_waves<LOGN, E>()))
ks_unit_kernel(LdModup<MODE == KS_ROTATE, 1> ld, HoistTab T, ModdownArgs A, ModdownHoist H, double *scratch,
               const double *__restrict__ tw_all, const double *__restrict__ itw_all, const DevConst *__restrict__ C)
{
    __shared__ __align__(16) double lds[2 * lds_doubles<LOGN>()];
    constexpr int TH = (1 << LOGN) / E, N = 1 << LOGN;
    constexpr bool GALOIS = MODE == KS_ROTATE;
    const int tid = threadIdx.x, k = C->k, L = C->L, dnum = C->dnum;
    auto at = [&](int it) { return GALOIS ? chunk_elem<E>(tid, it) : tid + it * TH; };
    uint64_t raw[E][1];
    auto fetch = [&](int b, int j) {
        const uint64_t *e = ld.src + (size_t)b * ld.unit_stride + ((size_t)j << LOGN);
#pragma unroll
        for (int it = 0; it < E; it++) raw[it][0] = GALOIS ? at32(e, at(it)) : at_lane(e + it * TH, tid);
    };
    fetch(blockIdx.x, 0);
    for (int b = blockIdx.x; b < A.batch; b += (int)gridDim.x) {
        const int b_next = b + (int)gridDim.x < A.batch ? b + (int)gridDim.x : b;
        double *keep = scratch + ((size_t)(2 * b) << LOGN);
        for (int step = 0; step < L; step++) {
            const int r = step ? step - 1 : k;
            const ModD m = C->mod[r];
            const double *tw = tw_all + ((size_t)r << LOGN), *itw = itw_all + ((size_t)r << LOGN);
            double s[2 * E], y[2 * E];
#pragma unroll
            for (int it = 0; it < 2 * E; it++) s[it] = 0.0;
            for (int j = 0; j < dnum; j++) {
                double x[E];
                const int row = (b * dnum + j) * L + r;
#pragma unroll
                for (int it = 0; it < E; it++) x[it] = ld.finish(raw[it], row, at(it), m, C);
                fetch(j + 1 < dnum || step + 1 < L ? b : b_next, j + 1 < dnum ? j + 1 : 0);
                lds_barrier();      // the previous reads of other waves' elements
                if constexpr (MODE == KS_PLAIN) {
                    int tk = tid;
                    asm volatile("" : "+v"(tk));
                    DigitKeys<LOGN, E> keys(T.key[0] + ((size_t)(2 * j * L + r) << LOGN), (size_t)L << LOGN, tk);
                    fwd_row<LOGN, E, false>(lds, x, x, tid, tw, m, [&] { keys.ask(0); });
                    if (dnum > 3) {     // as in ks_row_kernel
#pragma unroll
                        for (int it = 0; it < E; it++) x[it] = red(x[it], m);
                    }
                    keys.add(x, m, s, s + E);
                    continue;
                }
                if constexpr (GALOIS) {
#pragma unroll
                    for (int it = 0; it < E; it++) lds[pad(ld.place(at(it), N))] = x[it];
                    lds_barrier();
                }
                fwd_row<LOGN, E, GALOIS>(lds, x, x, tid, tw, m);
                int tk = tid;
                asm volatile("" : "+v"(tk));
                if constexpr (GALOIS) {
                    const double *k0 = T.key[0] + ((size_t)(2 * j * L + r) << LOGN), *k1 = k0 + ((size_t)L << LOGN);
                    if (dnum > 3) {     // as in ks_row_kernel
#pragma unroll
                        for (int it = 0; it < E; it++) x[it] = red(x[it], m);
                    }
#pragma unroll
                    for (int it = 0; it < E; it++) {
                        const int idx = chunk_elem<E>(tk, it);
                        s[it] += mulmod(x[it], at32(k0, idx), m);
                        s[E + it] += mulmod(x[it], at32(k1, idx), m);
                    }
                } else {
#pragma unroll
                    for (int it = 0; it < E; it += 2)
                        pair_at(lds, pad(chunk_elem<E>(tid, it))) = make_double2(red(x[it], m), red(x[it + 1], m));
                    lds_barrier();
                    sum_digit<LOGN, E, 2>(lds, T, H.n_sum, j, r, L, tk, m, s);
                }
            }
            const uint64_t *own_rows = (MODE == KS_ROTATE ? A.acc_add + (size_t)b * A.acc_stride
                                                          : A.add + (size_t)b * A.add_stride) + ((size_t)r << LOGN);
            const uint64_t *c0 = A.add + (size_t)b * A.add_stride + ((size_t)r << LOGN);
            uint64_t *out = A.out + (size_t)b * A.out_stride + ((size_t)r << LOGN);
            const size_t comp = (size_t)k << LOGN;
            const bool adds = MODE != KS_ROTATE || A.accumulate;
            // residues modulo the special prime, addends
            double xs[2 * E];
            uint64_t own[E];
#pragma unroll
            for (int it = 0; it < E; it++) xs[it] = xs[E + it] = 0.0, own[it] = 0;
            auto ask_own = [&](int c, int tk) {
                if (adds) {
#pragma unroll
                    for (int it = 0; it < E; it++) own[it] = at_lane(own_rows + c * comp + it * TH, tk);
                }
            };
            auto ask_xs = [&](int c, int tk) {
#pragma unroll
                for (int it = 0; it < E; it++) xs[c * E + it] = at_lane(keep + ((size_t)c << LOGN) + it * TH, tk);
            };
            // (rotations have no registers for them before the transform is done)
            auto ask = [&] {
                if (!step || MODE == KS_ROTATE) return;
                int tk = tid;
                asm volatile("" : "+v"(tk));
                ask_xs(0, tk);
                ask_xs(1, tk);
                ask_own(0, tk);
            };
            if (MODE == KS_SUM) lds_barrier();
            inv_row<LOGN, E, false, (MODE == KS_SUM ? hundredths(DotSum::OUT) : 0), 2>(lds, s, StRegs{y}, 0, tid, itw, m, r, C, 0, ask);
#pragma unroll
            for (int c = 0; c < 2; c++) {
                int tk = tid;
                asm volatile("" : "+v"(tk));
                if (!step) {        // centred residues modulo the special prime; every thread reads its own back
#pragma unroll
                    for (int it = 0; it < E; it++) put_lane(keep + ((size_t)c << LOGN) + it * TH, tk, red(y[c * E + it], m));
                    continue;
                }
                const size_t crow = c * comp;
                if (MODE == KS_ROTATE) ask_xs(c, tk);
                if (c || MODE == KS_ROTATE) ask_own(c, tk);
                double v[E];
#pragma unroll
                for (int it = 0; it < E; it++) v[it] = mulmod(y[c * E + it] - xs[c * E + it], C->Pinv_q[r], m);
                if (MODE != KS_PLAIN && c == 0) {
                    uint64_t w[E];
                    if (MODE == KS_ROTATE) {
#pragma unroll
                        for (int it = 0; it < E; it++) w[it] = at_lane(c0 + it * TH, tk);
                    }
                    lds_barrier();
#pragma unroll
                    for (int it = 0; it < E; it++) lds[tk + it * TH] = u64_to_f64(MODE == KS_ROTATE ? w[it] : own[it]);
                    lds_barrier();
                    const int n_sum = MODE == KS_SUM ? H.n_sum : 1;
                    for (int i = 0; i < n_sum; i++) {
                        // terms are canonical up to their sign: four of them between two reductions
                        const uint32_t ginv = MODE == KS_SUM ? H.ginv[i] : A.galois, e0 = (uint32_t)tk * ginv;
#pragma unroll
                        for (int it = 0; it < E; it++) {
                            const uint32_t e = e0 + (uint32_t)(it * TH) * ginv;
                            v[it] = signed_add(v[it], lds[e & (N - 1)], e << (31 - LOGN));
                        }
                        if (MODE == KS_SUM && (i & 3) == 3) {
#pragma unroll
                            for (int it = 0; it < E; it++) v[it] = red(v[it], m);
                        }
                    }
                }
#pragma unroll
                for (int it = 0; it < E; it++) {
                    if (adds) v[it] += u64_to_f64(own[it]);
                    put_lane(out + crow + it * TH, tk, f64_to_u64(canon(v[it], m)));
                }
            }
        }
    }
}

// The sum of a series of rotations of every ciphertext of a batch, as key-switch accumulators in
// transform order: acc[b][c][r] = sum_i sum_j digit_j[b][r][pi_{g_i}(.)] * key_i[j][c][r].  Summing
// before the inverse transform and the division by P costs one inverse transform and one mod-down
// per ciphertext instead of one per rotation.
//
// A thread owns one evaluation point of U ciphertexts, both components: a digit value is used for both
// components and a key value for U ciphertexts, (2 + U) / (2 U) operands per product where the inverse
// transform that formed the sum in its loader (one row per workgroup) read two; what bounds this is
// the rate at which a compute unit takes operands in from L2.  The products are not reduced one
// by one: with residues split as 2^25 hi + lo, hi hi', lo lo' and (hi + lo)(hi' + lo') accumulate
// exactly in 64-bit integers over all terms (at most 128 * 6 of them, each below 2^53) by three
// 32 x 32 + 64 multiply-adds, which run at the FP64 rate here, and one modular reduction ends it.
// N = 8192, 7 rotations, with the inverse transforms: 48 ciphertexts 77 -> 54 us, 12: 33 -> 20 us,
// one: 32 -> 14 us.
// AHEAD: a rotation's words are asked for while those of the one before are multiplied, its key's address and Galois element read one rotation sooner
// still (the dispatch says where).
// block blk of nblk
template <int DNUM, int U, bool AHEAD>
__device__ __forceinline__ void ks_sum_block(int blk, int nblk, const uint64_t *__restrict__ dig, const HoistTab &T, int n_rot, double *__restrict__ acc,
                                             int batch, const DevConst *__restrict__ C)
{
    const int logn = C->logn, L = C->L, chunks = (1 << logn) / PW_THREADS;
    // Logical order: prime, ciphertext group, chunk of the row (fastest); XCD x takes the x-th eighth of
    // it.  The gathers of a digit row then stay on one XCD, and an XCD works with the keys of one or
    // two primes.  (chunks is a multiple of 8.)
    const int per_xcd = nblk >> 3;
    const int lg = (blk & 7) * per_xcd + (blk >> 3);
    const int groups = (batch + U - 1) / U;
    const int idx = (lg % chunks) * PW_THREADS + (int)threadIdx.x;
    const int ug = lg / chunks % groups, r = lg / (chunks * groups);
    const uint64_t *d[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
        const int b = ug * U + u < batch ? ug * U + u : batch - 1;      // a last group may be short
        d[u] = dig + (((size_t)b * DNUM * L + r) << logn);
    }
    const size_t row = (size_t)L << logn, key_off = ((size_t)r << logn) + idx;
    const uint32_t e0 = 2u * (__brev((uint32_t)idx) >> (32 - logn)) + 1u;
    const ModD m = C->mod[r];
    uint64_t lo[U][2], mid[U][2], hi[U][2];
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
        for (int c = 0; c < 2; c++) lo[u][c] = mid[u][c] = hi[u][c] = 0;
    auto load = [&](uint32_t g, const double *key, uint64_t (&kv)[DNUM][2], uint64_t (&dv)[U][DNUM]) {
        const uint32_t e = (e0 * g) & ((2u << logn) - 1u);
        const int sidx = (int)(__brev(e >> 1) >> (32 - logn));
        const double *kb = key + key_off;
#pragma unroll
        for (int j = 0; j < DNUM; j++)
#pragma unroll
            for (int c = 0; c < 2; c++) kv[j][c] = f64_bits(kb[(size_t)(j * 2 + c) * row]);
#pragma unroll
        for (int u = 0; u < U; u++)
#pragma unroll
            for (int j = 0; j < DNUM; j++) dv[u][j] = d[u][(size_t)j * row + sidx];
    };
    auto use = [&](const uint64_t (&kv)[DNUM][2], const uint64_t (&dv)[U][DNUM]) {
#pragma unroll
        for (int j = 0; j < DNUM; j++) {
            uint32_t kl[2], kh[2];
#pragma unroll
            for (int c = 0; c < 2; c++) {
                const uint64_t q = f64_to_u64(bits_f64(kv[j][c]) + m.p);     // positive, below 2^51
                kl[c] = (uint32_t)q & 0x1FFFFFFu;
                kh[c] = (uint32_t)(q >> 25);
            }
#pragma unroll
            for (int u = 0; u < U; u++) {
                const uint32_t dl = (uint32_t)dv[u][j] & 0x1FFFFFFu, dh = (uint32_t)(dv[u][j] >> 25);
#pragma unroll
                for (int c = 0; c < 2; c++) {
                    lo[u][c] += (uint64_t)dl * kl[c];
                    hi[u][c] += (uint64_t)dh * kh[c];
                    mid[u][c] += (uint64_t)(dl + dh) * (kl[c] + kh[c]);
                }
            }
        }
    };
    if constexpr (AHEAD) {
        uint32_t g = T.g[0];
        const double *key = T.key[0];
        uint64_t kv[2][DNUM][2], dv[2][U][DNUM];
        auto ask = [&](int w, int next) {
            load(g, key, kv[w], dv[w]);
            next = next < n_rot ? next : n_rot - 1;
            g = T.g[next];
            key = T.key[next];
        };
        int i = 0;
        // an even number's first one goes by itself, so that nothing is asked for in vain
        if (n_rot % 2 == 0) {
            ask(0, 1);
            use(kv[0], dv[0]);
            i = 1;
        }
        ask(0, i + 1);
        for (; i + 1 < n_rot; i += 2) {
            ask(1, i + 2);
            __builtin_amdgcn_sched_barrier(0);
            use(kv[0], dv[0]);
            ask(0, i + 3);
            __builtin_amdgcn_sched_barrier(0);
            use(kv[1], dv[1]);
        }
        if (i < n_rot) use(kv[0], dv[0]);
    } else {
        for (int i = 0; i < n_rot; i++) {
            uint64_t kv[DNUM][2], dv[U][DNUM];
            load(T.g[i], T.key[i], kv, dv);
            use(kv, dv);
        }
    }
    const double t50 = C->two50[r], t81 = C->two81[r];
#pragma unroll
    for (int u = 0; u < U; u++) {
        if (ug * U + u >= batch) break;
#pragma unroll
        for (int c = 0; c < 2; c++) {
            // lo + 2^25 (mid - lo - hi) + 2^50 hi with the carries moved up, then modulo the prime
            const uint64_t x = (lo[u][c] >> 25) + (mid[u][c] - lo[u][c] - hi[u][c]);
            const uint64_t low = (lo[u][c] & 0x1FFFFFFu) | ((x & 0x1FFFFFFu) << 25);
            const uint64_t top = hi[u][c] + (x >> 25);
            const double v = u64_to_f64(low) + mulmod((double)((uint32_t)top & 0x7FFFFFFFu), t50, m) +
                             mulmod((double)(uint32_t)(top >> 31), t81, m);
            acc[(((size_t)((ug * U + u) * 2 + c) * L + r) << logn) + idx] = v;
        }
    }
}

template <int DNUM, int U, bool AHEAD>
__global__ void __launch_bounds__(PW_THREADS)
ks_sum_kernel(const uint64_t *__restrict__ dig, HoistTab T, int n_rot, double *__restrict__ acc, int batch,
              const DevConst *__restrict__ C)
{
    ks_sum_block<DNUM, U, AHEAD>((int)blockIdx.x, (int)gridDim.x, dig, T, n_rot, acc, batch, C);
}

// Block blk of a mod-down that a mod-up took ahead of it (LdModupDown): THREADS pairs of coefficients of one row (unit, component, prime) of
//   out = in + u (+ sum_r sigma_r(c0), component 0),
// the permuted coefficients gathered from L2, four rotations' together; it runs beside longer blocks.
template <int THREADS>
__device__ __forceinline__ void down_block(int blk, const ModdownArgs &A, const ModdownHoist &H, const DevConst *__restrict__ C)
{
    const int logn = C->logn, k = C->k, chunks = (1 << logn) / (2 * THREADS);
    const int row = blk / chunks, n = (blk % chunks * THREADS + (int)threadIdx.x) * 2, i = row % k, bc = row / k, b = bc >> 1, c = bc & 1;
    const uint32_t mask = (1u << logn) - 1u;
    const ModD m = C->mod[i];
    const uint64_t *in = A.add + (size_t)b * A.add_stride + ((size_t)(c * k + i) << logn);
    const double *a = A.acc + (((size_t)bc * C->L) << logn) + n;
    const double2 xp = *reinterpret_cast<const double2 *>(a + ((size_t)k << logn)), ap = *reinterpret_cast<const double2 *>(a + ((size_t)i << logn));
    const ulonglong2 own = *reinterpret_cast<const ulonglong2 *>(in + n);
    double v0 = mulmod(ap.x - red(xp.x, C->mod[k]), C->Pinv_q[i], m), v1 = mulmod(ap.y - red(xp.y, C->mod[k]), C->Pinv_q[i], m);
    const int n_sum = c ? 0 : H.n_sum;
    for (int r0 = 0; r0 < n_sum; r0 += 4) {
        // terms are canonical up to their sign: four of them between two reductions
        uint64_t w[4][2];
        uint32_t e[4][2];
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const uint32_t g = H.ginv[r0 + r < n_sum ? r0 + r : 0];
            e[r][0] = (uint32_t)n * g;
            e[r][1] = e[r][0] + g;
#pragma unroll
            for (int h = 0; h < 2; h++) w[r][h] = in[e[r][h] & mask];
        }
#pragma unroll
        for (int r = 0; r < 4; r++)
            if (r0 + r < n_sum) {
                v0 = signed_add(v0, u64_to_f64(w[r][0]), e[r][0] << (31 - logn));
                v1 = signed_add(v1, u64_to_f64(w[r][1]), e[r][1] << (31 - logn));
            }
        v0 = red(v0, m);
        v1 = red(v1, m);
    }
    uint64_t *o = A.out + (size_t)b * A.out_stride + ((size_t)(c * k + i) << logn) + n;
    *reinterpret_cast<ulonglong2 *>(o) =
        make_ulonglong2(f64_to_u64(canon(v0 + u64_to_f64(own.x), m)), f64_to_u64(canon(v1 + u64_to_f64(own.y), m)));
}

// The same, and behind its n_sums blocks those of the mod-down before.  A series of dependent key switches of few units is bound by its launches, of
// which this takes one away for each.
template <int DNUM>
__global__ void __launch_bounds__(PW_THREADS)
ks_sum_after_kernel(const uint64_t *__restrict__ dig, HoistTab T, int n_rot, double *__restrict__ acc, int batch, int n_sums,
                    ModdownArgs A, ModdownHoist H, const DevConst *__restrict__ C)
{
    if ((int)blockIdx.x < n_sums) ks_sum_block<DNUM, 1, true>((int)blockIdx.x, n_sums, dig, T, n_rot, acc, batch, C);
    else down_block<PW_THREADS>((int)blockIdx.x - n_sums, A, H, C);
}
// One rotation's, or a relinearisation's, inner product in the loader of its inverse transform, nwg rows
template <int LOGN, int E, int DNUM>
__global__ void __launch_bounds__((1 << LOGN) / E, (min_waves<LOGN, E>()))
ks_inner_after_kernel(LdInvKsInner<DNUM> ld, StInvF64 st, const double *__restrict__ itw_all, int nwg, ModdownArgs A, ModdownHoist H,
                      const DevConst *__restrict__ C)
{
    __shared__ __align__(16) double lds[lds_doubles<LOGN>()];
    if ((int)blockIdx.x < nwg) inv_rows<LOGN, E>(lds, (int)blockIdx.x, nwg, ld, st, itw_all, C, nwg);
    else down_block<(1 << LOGN) / E>((int)blockIdx.x - nwg, A, H, C);
}

// ciphertext u of `src` (src_stride words apart) to dst + u * dst_stride, two words per thread
__global__ void __launch_bounds__(PW_THREADS)
copy_kernel(const uint64_t *__restrict__ src, size_t src_stride, uint64_t *__restrict__ dst, size_t dst_stride, int blocks_per_ct)
{
    const int u = (int)blockIdx.x / blocks_per_ct, at = (((int)blockIdx.x % blocks_per_ct) * PW_THREADS + (int)threadIdx.x) * 2;
    *reinterpret_cast<ulonglong2 *>(dst + u * dst_stride + at) = *reinterpret_cast<const ulonglong2 *>(src + u * src_stride + at);
}

// out = a + b over `rows` rows of N residues, row w modulo q_(w % k)
__global__ void __launch_bounds__(PW_THREADS)
add_kernel(const uint64_t *__restrict__ a, const uint64_t *__restrict__ b, uint64_t *__restrict__ out,
           int rows, const DevConst *__restrict__ C)
{
    const int logn = C->logn, N = 1 << logn;
    const size_t gid = (size_t)blockIdx.x * PW_THREADS + threadIdx.x;
    const int row = (int)(gid >> logn);
    if (row >= rows) return;
    (void)N;
    const ModD m = C->mod[row % C->k];
    out[gid] = f64_to_u64(addmod_canon(u64_to_f64(a[gid]), u64_to_f64(b[gid]), m));
}

// out[b] = in[b] + sign * floor(Q/t) * pt  (the plaintext enters component 0 only; component 1 is
// copied): rows = batch * 2 * k, pt[(b % p_mod)][N] coefficients in [0, t)
__global__ void __launch_bounds__(PW_THREADS)
add_plain_kernel(const uint64_t *__restrict__ in, const uint64_t *__restrict__ pt, uint64_t *__restrict__ out,
                 int batch, int p_mod, int negative, const DevConst *__restrict__ C)
{
    const int logn = C->logn, N = 1 << logn, k = C->k;
    const size_t gid = (size_t)blockIdx.x * PW_THREADS + threadIdx.x;
    const int n = (int)(gid & (N - 1));
    const int row = (int)(gid >> logn);
    if (row >= batch * 2 * k) return;
    const int i = row % k, c = (row / k) & 1, b = row / (2 * k);
    double v = u64_to_f64(in[gid]);
    if (c == 0) {
        const ModD m = C->mod[i];
        const double d = canon(mulmod(u64_to_f64(pt[((size_t)(b % p_mod) << logn) + n]), C->delta_q[i], m), m);
        v = negative ? (v >= d ? v - d : v - d + m.p) : addmod_canon(v, d, m);
    }
    out[gid] = f64_to_u64(v);
}

// out[g][e] = sum_{c < group} in[g*group + c][e] over rows*N elements per unit (row w mod q_(w%k))
__global__ void __launch_bounds__(PW_THREADS)
sum_groups_kernel(const uint64_t *__restrict__ in, uint64_t *__restrict__ out, int groups, int group,
                  int rows, const DevConst *__restrict__ C)
{
    const int logn = C->logn;
    const size_t per = (size_t)rows << logn;
    const size_t gid = (size_t)blockIdx.x * PW_THREADS + threadIdx.x;
    if (gid >= per * (size_t)groups) return;
    const size_t g = gid / per, e = gid % per;
    const ModD m = C->mod[(int)(e >> logn) % C->k];
    double s = u64_to_f64(in[(g * group) * per + e]);
    for (int c = 1; c < group; c++) s = addmod_canon(s, u64_to_f64(in[(g * group + c) * per + e]), m);
    out[gid] = f64_to_u64(s);
}

// Exchange micro-benchmark: the wave-local regrouping a transform pass boundary needs when the
// next stage pairs elements 32 lanes apart.  Every lane holds 16 doubles; one exchange hands the
// upper 8 of lanes 0-31 to lanes 32-63 in return for their lower 8 (afterwards a lane holds both
// halves of 8 butterflies).  kind 0: through the wave's own region of LDS (8 stores, wave-level
// ordering, 8 loads per lane); kind 1: v_permlane32_swap on the 32-bit halves (16 instructions per
// lane, no memory).  One add per held double between exchanges keeps the values moving.
typedef unsigned cg_uint2v __attribute__((ext_vector_type(2)));
__global__ void __launch_bounds__(1024)
bench_exchange_kernel(int kind, uint32_t iters, double *__restrict__ out)
{
    __shared__ double lds[16 * 64 * 8];
    const int tid = threadIdx.x, lane = tid & 63;
    double *mine = lds + (tid >> 6) * (64 * 8);
    double v[16];
#pragma unroll
    for (int k = 0; k < 16; k++) v[k] = (double)(tid * 16 + k);
    for (uint32_t i = 0; i < iters; i++) {
        if (kind == 0) {
            // a lane gives away its upper half (lanes 0-31) or its lower half (lanes 32-63)
#pragma unroll
            for (int k = 0; k < 8; k++) mine[k * 64 + lane] = lane < 32 ? v[8 + k] : v[k];
            wave_sync();
#pragma unroll
            for (int k = 0; k < 8; k++) {
                const double got = mine[k * 64 + (lane ^ 32)];
                if (lane < 32) v[8 + k] = got;
                else v[k] = got;
            }
            wave_sync();
        } else {
#pragma unroll
            for (int k = 0; k < 8; k++) {
                uint64_t a = f64_bits(v[k]), b = f64_bits(v[8 + k]);
                // upper 32 lanes of the first operand <-> lower 32 lanes of the second
                const cg_uint2v lo = __builtin_amdgcn_permlane32_swap((unsigned)a, (unsigned)b, false, false);
                const cg_uint2v hi = __builtin_amdgcn_permlane32_swap((unsigned)(a >> 32), (unsigned)(b >> 32), false, false);
                v[k] = bits_f64(((uint64_t)hi.x << 32) | lo.x);
                v[8 + k] = bits_f64(((uint64_t)hi.y << 32) | lo.y);
            }
        }
#pragma unroll
        for (int k = 0; k < 16; k++) v[k] += 1.0;
    }
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 16; k++) s += v[k] * (double)(k + 1);
    out[(size_t)blockIdx.x * blockDim.x + tid] = s;
}

// arithmetic micro-benchmark: `iters` dependent products per lane
__global__ void __launch_bounds__(PW_THREADS)
bench_modmul_kernel(int kind, uint32_t n_lanes, uint32_t iters, uint64_t *__restrict__ out, ModD md, ModI mi)
{
    const uint32_t gid = blockIdx.x * PW_THREADS + threadIdx.x;
    if (gid >= n_lanes) return;
    const uint64_t x0 = (0x9E3779B97F4A7C15ull * (gid + 1)) % mi.q;
    const uint64_t w0 = (0xD1B54A32D192ED03ull * (gid + 7)) % mi.q;
    if (kind == 0) {
        double x = u64_to_f64(x0), y = u64_to_f64(w0);
        const double w = u64_to_f64(w0);
        for (uint32_t i = 0; i < iters; i++) {
            x = mulmod(x, w, md);
            y = mulmod(y, x, md);
        }
        out[gid] = f64_to_u64(canon(x, md)) ^ f64_to_u64(canon(y, md));
    } else {
        uint64_t x = x0, y = w0;
        for (uint32_t i = 0; i < iters; i++) {
            x = mulmod_barrett(x, w0, mi);
            y = mulmod_barrett(y, x, mi);
        }
        out[gid] = x ^ y;
    }
}

}  // namespace cg
