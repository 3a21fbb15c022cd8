// C ABI of the library (see include/cryptogen.h): context set-up on the host,
// argument checks, and the launch sequences of the evaluator operations.
#include "../../include/cryptogen.h"
#include "../../include/cryptogen_bench.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <tuple>
#include <unordered_map>
#include <vector>

#include "kernels.hpp"

using namespace cg;

typedef unsigned __int128 u128;

// Workspace of cg_mul_relin_static, the entry point for callers that cannot allocate: device
// memory that belongs to the loaded library itself (one copy per GPU, held until the process
// ends).  In host code this name is only a handle for the runtime's symbol look-up; the address the
// kernels get is the one hipGetSymbolAddress returns on the device in question, kept below.
__device__ __align__(256) unsigned char scratch[CG_STATIC_SCRATCH_BYTES];
static constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void *g_scratch_ptr[kMaxDevices];   // per device; null until a context was created there
// the array's address on `device`, which must be the current device
static int static_scratch_address(int device, void **out)
{
    if (device < 0 || device >= kMaxDevices) return CG_EINVAL;
    std::lock_guard<std::mutex> g(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return CG_EHIP;
        g_scratch_ptr[device] = p;
    }
    *out = g_scratch_ptr[device];
    return CG_OK;
}

// Side streams of the one-call decode step.  Calls on the default stream of a GPU use one pair for all of its
// contexts, calls on any other stream a pair of the context's own.
// Why a common pair: the runtime maps streams onto four hardware queues, and with a pair per context the pairs of the
// third and later contexts of a process came to lie on the queue of the caller's own stream, so that the step's
// branches ran one after the other (12 heads, 512 tokens, N = 8192, four contexts alive: 0.725 ms a step, against 0.515
// with one pair).
// Why only there: a branch waits for everything ahead of it on its side stream, so a common pair puts a call behind
// whatever earlier users' fork events wait for.  On one and the same stream that is no new order: the
// stream itself has the later call wait for the earlier one.  Across streams it would be (a step on an idle stream
// held up, or blocked for good, by what another context's stream waits for), and a capture would take in
// other callers' work.  The default stream cannot be captured, is there once per GPU and never destroyed.
// The common pair is created by a device's first context and destroyed with its last.
struct SidePair {
    hipStream_t stream[2];
    int users;
};
static std::mutex g_side_mu;
static SidePair g_side[kMaxDevices];
static void destroy_pair(hipStream_t *p)
{
    for (int i = 0; i < 2; i++) {
        if (p[i]) (void)hipStreamDestroy(p[i]);
        p[i] = nullptr;
    }
}
static bool create_pair(hipStream_t *p)
{
    for (int i = 0; i < 2; i++)
        if (hipStreamCreateWithFlags(&p[i], hipStreamNonBlocking) != hipSuccess) {
            p[i] = nullptr;
            destroy_pair(p);
            return false;
        }
    return true;
}
static bool side_acquire(int device, hipStream_t *out)
{
    if (device < 0 || device >= kMaxDevices) return false;
    std::lock_guard<std::mutex> g(g_side_mu);
    SidePair &sp = g_side[device];
    if (sp.users == 0 && !create_pair(sp.stream)) return false;
    sp.users++;
    for (int i = 0; i < 2; i++) out[i] = sp.stream[i];
    return true;
}
static void side_release(int device)
{
    std::lock_guard<std::mutex> g(g_side_mu);
    SidePair &sp = g_side[device];
    if (--sp.users == 0) destroy_pair(sp.stream);
}

// ---------------------------------------------------------------------------
// host integer helpers (set-up only)
// ---------------------------------------------------------------------------
static uint64_t h_mul(uint64_t a, uint64_t b, uint64_t m) { return (uint64_t)((u128)a * b % m); }
static uint64_t h_pow(uint64_t a, uint64_t e, uint64_t m)
{
    uint64_t r = 1;
    a %= m;
    for (; e; e >>= 1, a = h_mul(a, a, m))
        if (e & 1) r = h_mul(r, a, m);
    return r;
}
static uint64_t h_inv(uint64_t a, uint64_t m) { return h_pow(a % m, m - 2, m); }
// Primality below 2^64 by strong-probable-prime tests to the seven bases of Sinclair's set, which
// has no composite below 2^64 passing all of them; trial division first, to leave early.
static bool h_is_prime(uint64_t n)
{
    if (n < 4) return n == 2 || n == 3;
    if (!(n & 1)) return false;
    for (uint64_t f = 3; f < 64; f += 2) {
        if (n == f) return true;
        if (n % f == 0) return false;
    }
    const int two = __builtin_ctzll(n - 1);
    const uint64_t odd = (n - 1) >> two;
    static const uint64_t bases[7] = {2, 325, 9375, 28178, 450775, 9780504, 1795265022};
    for (uint64_t b : bases) {
        uint64_t y = h_pow(b % n, odd, n);
        if (y <= 1 || y == n - 1) continue;            // b = 0 mod n gives y = 0: no witness
        int sq = 1;
        while (sq < two && y != n - 1) { y = h_mul(y, y, n); sq++; }
        if (y != n - 1) return false;
    }
    return true;
}
// smallest primitive 2N-th root of unity mod p (the convention of cg_ntt_forward): any primitive
// root, then the minimum over its N odd powers, which are all the primitive 2N-th roots
static uint64_t h_min_root(uint64_t p, uint64_t n)
{
    const uint64_t cof = (p - 1) / (2 * n);
    uint64_t any = 0;
    for (uint64_t cand = 2; !any; cand++) {
        const uint64_t r = h_pow(cand, cof, p);      // order divides 2N; it is 2N iff r^N = -1
        if (h_pow(r, n, p) == p - 1) any = r;
    }
    const uint64_t step = h_mul(any, any, p);
    uint64_t lo = any, w = any;
    for (uint64_t i = 1; i < n; i++) {
        w = h_mul(w, step, p);
        lo = w < lo ? w : lo;
    }
    return lo;
}
static uint32_t h_bitrev(uint32_t x, int bits)
{
    uint32_t r = 0;
    for (int i = 0; i < bits; i++) { r = (r << 1) | (x & 1); x >>= 1; }
    return r;
}
static double h_centred(uint64_t x, uint64_t p) { return x > p / 2 ? -(double)(p - x) : (double)x; }

// ---------------------------------------------------------------------------
// context
// ---------------------------------------------------------------------------
struct cg_ctx {
    int logn, N, k, nsp, alpha, dnum, l, L, KL, np;
    uint64_t t;
    uint64_t pr[MAXPR];
    DevConst hc;
    DevConst *dc;
    double *tw, *itw;     // [np][N] forward / inverse twiddles (centred doubles, bit-reversed order)
    double *tw2, *itw2;   // N = 16384: [np][2][N/2], those of the two half rows
    uint32_t *tab;        // scratch prime-index table for the public transform entry points
    uint32_t tab_cap;
    int device, n_cu;
    void *static_ws;      // this device's copy of the library-owned scratch array
    // resident workgroups per compute unit of every transform-kernel instantiation this context
    // launches, keyed by the kernel's address: filled by cg_create (a dry pass over all launch
    // sequences), so that no launch has to ask the runtime; the lock covers a late first use
    std::mutex *occ_mu;
    std::unordered_map<const void *, int> *occ;
    bool dry;             // set-up pass: launches compute their grid and return without launching
    bool dry_units;                 // while dry: and of whole key switches
    bool dry_rows;                  // while dry: take the kernels of several transforms per workgroup
    int elems, elems_fwd; // elements per thread in the inverse / forward transform kernels (8 or 16)
    // workspace limbs (N * 8 bytes) per unit
    int ws_total;
    // side streams (default priority) and fork/join events for entry points that run independent branches side by
    // side: the device's pair for calls on its default stream, the context's own pair for calls on others
    hipStream_t side_default[2], side_own[2];
    hipEvent_t ev_fork, ev_join[2];
    // optional per-launch timing with HIP events (benchmark support)
    bool prof_on;
    uint32_t prof_n, prof_cap;
    hipEvent_t *prof_ev;      // 2 * prof_cap events
    uint8_t *prof_id;
    double *prof_bytes;
    double *prof_items;
};

// kernel classes for the timing facility
enum KernelId {
    KID_FWD_MULQ = 0, KID_FWD_MULB, KID_FWD_MODUP, KID_FWD_ROWS, KID_FWD_PLAIN,
    KID_INV_TENSOR, KID_INV_U64, KID_INV_MULPLAIN, KID_SCALE, KID_INV_KSINNER, KID_MODDOWN,
    KID_ADD, KID_SUM_GROUPS, KID_KSSUM, KID_MODDOWN_SUM, KID_INV_TENSORSUM, KID_MULPLAIN, KID_INV_F64, KID_KSROW, KID_MULROW, KID_KSSUMROW, KID_MULSUMROW, KID_FWD_MULEXT, KID_ROTROW, KID_KSUNIT, KID_LIFT, KID_FWD_HALF, KID_COPY, KID_KSSUMDOWN, KID_COUNT
};
static const char *const kKernelNames[KID_COUNT] = {
    "ntt_fwd<mul,q-rows>", "ntt_fwd<mul,aux-rows>", "ntt_fwd<modup>", "ntt_fwd<rows>",
    "ntt_fwd<plain>", "ntt_inv<tensor>", "ntt_inv<u64>", "ntt_inv<mul_plain>", "scale",
    "ntt_inv<ks_inner>", "moddown", "add", "sum_groups", "ks_sum", "moddown<sum>",
    "ntt_inv<tensor_sum>", "ntt_fwd_inv<mul_plain>", "ntt_inv<f64>", "ks_row", "mul_row", "ks_sum_row", "mul_sum_row", "ntt_fwd<mul,all-rows>", "rot_row", "ks_unit", "lift", "ntt_fwd<mul,half-rows>", "copy", "ks_sum_down"};

// Brackets one launch with two events when profiling is on.
struct ProfScope {
    cg_ctx *c;
    hipStream_t s;
    int slot;
    // items: residue rows a transform launch works through, batch units for a pointwise launch
    ProfScope(cg_ctx *c_, hipStream_t s_, int id, double bytes, double items) : c(c_), s(s_), slot(-1)
    {
        if (c->prof_on && c->prof_n < c->prof_cap) {
            slot = (int)c->prof_n++;
            c->prof_id[slot] = (uint8_t)id;
            c->prof_bytes[slot] = bytes;
            c->prof_items[slot] = items;
            (void)hipEventRecord(c->prof_ev[2 * slot], s);
        }
    }
    ~ProfScope()
    {
        if (slot >= 0) (void)hipEventRecord(c->prof_ev[2 * slot + 1], s);
    }
};

static void fill_conv(ConvTab &T, const uint64_t *pr, const int *sidx, int ns, const int *tidx, int nt)
{
    memset(&T, 0, sizeof(T));
    for (int i = 0; i < ns; i++)
        for (int j = i + 1; j < ns; j++) {
            const uint64_t si = pr[sidx[i]], sj = pr[sidx[j]];
            T.inv[i][j] = h_centred(h_inv(si % sj, sj), sj);
        }
    for (int j = 0; j < nt; j++) {
        const uint64_t tj = pr[tidx[j]];
        for (int i = 0; i < ns; i++) T.s_mod_t[i][j] = h_centred(pr[sidx[i]] % tj, tj);
    }
}

static bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
#define CG_REQUIRE(cond) do { if (!(cond)) return CG_EINVAL; } while (0)
#define CG_HIP(call) do { if ((call) != hipSuccess) return CG_EHIP; } while (0)
// Launch through the runtime's C entry point: its return value is this launch's own status, so an
// error that other code left pending in the thread is neither reported as ours nor cleared.
template <class... P, class... A>
static int launch_kernel(void (*kernel)(P...), dim3 grid, dim3 block, hipStream_t s, A... args)
{
    std::tuple<P...> pack{static_cast<P>(args)...};
    void *ptrs[sizeof...(P)];
    int i = 0;
    std::apply([&](auto &...e) { ((ptrs[i++] = static_cast<void *>(&e)), ...); }, pack);
    return hipLaunchKernel(reinterpret_cast<const void *>(kernel), grid, block, ptrs, 0, s) == hipSuccess ? CG_OK
                                                                                                         : CG_EHIP;
}

extern "C" const char *cg_strerror(int status)
{
    switch (status) {
    case CG_OK: return "ok";
    case CG_EINVAL: return "invalid argument";
    case CG_ENOMEM: return "out of device memory";
    case CG_EHIP: return "HIP runtime error";
    case CG_ESCRATCH: return "batch needs more scratch than the library's static array holds";
    default: return "unknown status";
    }
}

static int warm_launch_table(cg_ctx *c);

extern "C" int cg_create(cg_ctx **out, const cg_params *prm)
{
    CG_REQUIRE(out && prm && prm->q && prm->p);
    *out = nullptr;
    CG_REQUIRE(prm->log2n >= 12 && prm->log2n <= 14);
    CG_REQUIRE(prm->k >= 1 && prm->k <= 6 && prm->nsp >= 1 && prm->nsp <= 2);
    CG_REQUIRE(prm->alpha >= 1 && prm->alpha <= 2 && prm->k % prm->alpha == 0);
    // a digit of alpha primes against fewer special primes makes P smaller than Q_j by a whole prime:
    // every result would still match its definition, but a key switch would add noise of the size of
    // a prime and silently use up the decryption budget
    CG_REQUIRE(prm->alpha <= prm->nsp);
    CG_REQUIRE((prm->t & 1) && prm->t > 2 && prm->t < (1u << 20));
    const uint64_t N = 1ull << prm->log2n;
    cg_ctx *c = new (std::nothrow) cg_ctx();
    if (!c) return CG_ENOMEM;
    memset(c, 0, sizeof(*c));
    c->occ_mu = new (std::nothrow) std::mutex();
    c->occ = new (std::nothrow) std::unordered_map<const void *, int>();
    if (!c->occ_mu || !c->occ) { cg_destroy(c); return CG_ENOMEM; }
    c->logn = (int)prm->log2n; c->N = (int)N; c->k = (int)prm->k; c->nsp = (int)prm->nsp;
    c->alpha = (int)prm->alpha; c->dnum = c->k / c->alpha; c->t = prm->t;
    c->l = c->k + 1;
    c->elems = c->logn <= 13 ? 8 : 16;              // 1024 threads per row at N >= 8192, 512 at N = 4096
    c->elems_fwd = c->logn == 13 ? 16 : c->elems;   // two 512-thread workgroups per compute unit at N = 8192
    c->L = c->k + c->nsp;
    c->KL = c->k + c->l;
    int np = 0;
    uint64_t lowest = ~0ull;
    auto ok_prime = [&](uint64_t p) {
        if (!(p > (1ull << 40) && p < (1ull << 50) && p % (2 * N) == 1 && h_is_prime(p))) return false;
        for (int i = 0; i < np; i++) if (c->pr[i] == p) return false;
        return true;
    };
    for (uint32_t i = 0; i < prm->k + prm->nsp; i++) {
        const uint64_t p = i < prm->k ? prm->q[i] : prm->p[i - prm->k];
        if (!ok_prime(p) || p == prm->t) { cg_destroy(c); return CG_EINVAL; }
        c->pr[np++] = p;
        if (p < lowest) lowest = p;
    }
    // auxiliary basis for the tensor product: the special primes plus private primes
    // below every given prime, l = k + 1 in total
    uint64_t cand = lowest;
    while (np < c->k + c->l) {
        cand -= 2 * N;
        if (cand <= (1ull << 40)) { cg_destroy(c); return CG_EINVAL; }
        if (ok_prime(cand) && cand != prm->t) c->pr[np++] = cand;
    }
    c->np = np;
    // the scaled product round(t e / Q) is below t N Q in magnitude and must fit the centred
    // range of the auxiliary basis
    double lgQ = 0, lgB = 0;
    for (int i = 0; i < c->k; i++) lgQ += std::log2((double)c->pr[i]);
    for (int j = 0; j < c->l; j++) lgB += std::log2((double)c->pr[c->k + j]);
    if (!(lgB > lgQ + std::log2((double)c->t) + c->logn + 3)) { cg_destroy(c); return CG_EINVAL; }

    DevConst &H = c->hc;
    memset(&H, 0, sizeof(H));
    H.logn = c->logn; H.k = c->k; H.nsp = c->nsp; H.l = c->l; H.alpha = c->alpha; H.dnum = c->dnum;
    H.L = c->L; H.KL = c->KL; H.np = np; H.tmod = (double)c->t;
    std::vector<double> tw((size_t)np * N), itw((size_t)np * N);
    for (int r = 0; r < np; r++) {
        const uint64_t p = c->pr[r];
        H.mod[r].p = (double)p;
        H.mod[r].u = 1.0 / (double)p;
        const uint64_t psi = h_min_root(p, N);
        std::vector<uint64_t> pw(N);
        pw[0] = 1;
        for (uint64_t i = 1; i < N; i++) pw[i] = h_mul(pw[i - 1], psi, p);
        for (uint64_t j = 0; j < N; j++) {
            const uint64_t w = pw[h_bitrev((uint32_t)j, c->logn)];
            tw[(size_t)r * N + j] = h_centred(w, p);
            itw[(size_t)r * N + j] = h_centred(h_inv(w, p), p);
        }
        const uint64_t ninv = h_inv(N % p, p);
        H.ninv[r] = h_centred(ninv, p);
        H.t_ninv[r] = h_centred(h_mul(c->t % p, ninv, p), p);
        H.itw1_ninv[r] = h_centred(h_mul(h_inv(pw[h_bitrev(1, c->logn)], p), ninv, p), p);
    }
    std::vector<double> tw2, itw2;
    if (c->logn == 14) {
        // factors of half h: those of the whole row's stages from the second on, blocks h 2^s ... of stage s + 1
        const size_t half = N / 2;
        tw2.resize((size_t)np * N);
        itw2.resize((size_t)np * N);
        for (int r = 0; r < np; r++) {
            const double *t = &tw[(size_t)r * N], *it = &itw[(size_t)r * N];
            for (size_t h = 0; h < 2; h++) {
                double *t2 = &tw2[(size_t)r * N + h * half], *it2 = &itw2[(size_t)r * N + h * half];
                for (size_t w = 1; w < half; w *= 2)
                    for (size_t j = 0; j < w; j++) {
                        t2[w + j] = t[2 * w + h * w + j];
                        it2[w + j] = it[2 * w + h * w + j];
                    }
            }
            H.tw1[r] = t[1];
            H.itw1[r] = it[1];
        }
    }
    for (int r = 0; r < np; r++) {
        H.two50[r] = h_centred(h_pow(2, 50, c->pr[r]), c->pr[r]);
        H.two81[r] = h_centred(h_pow(2, 81, c->pr[r]), c->pr[r]);
    }
    int qi[MAXS], bi[MAXS], all[MAXT], sp[MAXS];
    for (int i = 0; i < c->k; i++) qi[i] = i;
    for (int j = 0; j < c->l; j++) bi[j] = c->k + j;
    for (int r = 0; r < c->L; r++) all[r] = r;
    for (int s = 0; s < c->nsp; s++) sp[s] = c->k + s;
    fill_conv(H.q2b, c->pr, qi, c->k, bi, c->l);
    fill_conv(H.b2q, c->pr, bi, c->l, qi, c->k);
    for (int j = 0; j < c->l; j++) {
        const uint64_t b = c->pr[c->k + j];
        uint64_t prod = 1;
        for (int i = 0; i < c->k; i++) prod = h_mul(prod, c->pr[i] % b, b);
        H.Qinv_b[j] = h_centred(h_inv(prod, b), b);
    }
    for (int j = 0; j < c->dnum; j++) fill_conv(H.dig[j], c->pr, qi + j * c->alpha, c->alpha, all, c->L);
    fill_conv(H.p2q, c->pr, sp, c->nsp, qi, c->k);
    for (int r = 0; r < c->k; r++) {
        const uint64_t m = c->pr[r];
        uint64_t P = 1;
        for (int s = 0; s < c->nsp; s++) P = h_mul(P, c->pr[c->k + s] % m, m);
        H.Pinv_q[r] = h_centred(h_inv(P, m), m);
    }
    {
        // floor(Q/t) = (Q - (Q mod t)) / t, and Q = 0 modulo q_i: floor(Q/t) = -(Q mod t) t^-1 (mod q_i)
        uint64_t q_mod_t = 1;
        for (int j = 0; j < c->k; j++) q_mod_t = h_mul(q_mod_t, c->pr[j] % c->t, c->t);
        for (int i = 0; i < c->k; i++) {
            const uint64_t m = c->pr[i];
            const uint64_t d = h_mul(m - q_mod_t % m, h_inv(c->t % m, m), m);
            H.delta_q[i] = h_centred(d % m, m);
        }
    }
    // workspace limbs per unit: three ciphertext temporaries (3k + 2k + 2k) plus the larger of the
    // tensor-product and key-switch scratch areas (kept separate for simplicity)
    c->ws_total = 7 * c->k + (4 * c->l + 7 * c->KL) + (c->dnum * c->L + 2 * c->L);

    if (hipGetDevice(&c->device) != hipSuccess ||
        hipDeviceGetAttribute(&c->n_cu, hipDeviceAttributeMultiprocessorCount, c->device) != hipSuccess ||
        c->n_cu < 1) {
        cg_destroy(c);
        return CG_EHIP;
    }
    {
        const int src = static_scratch_address(c->device, &c->static_ws);
        if (src != CG_OK) { cg_destroy(c); return src; }
    }
    const size_t tbytes = (size_t)np * N * sizeof(double);
    c->tab_cap = 1u << 16;
    if (hipMalloc(&c->dc, sizeof(DevConst)) != hipSuccess || hipMalloc(&c->tw, tbytes) != hipSuccess ||
        hipMalloc(&c->itw, tbytes) != hipSuccess ||
        (!tw2.empty() && (hipMalloc(&c->tw2, tbytes) != hipSuccess || hipMalloc(&c->itw2, tbytes) != hipSuccess)) ||
        hipMalloc(&c->tab, c->tab_cap * sizeof(uint32_t)) != hipSuccess) {
        cg_destroy(c);
        return CG_ENOMEM;
    }
    if (hipMemcpy(c->dc, &H, sizeof(DevConst), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(c->tw, tw.data(), tbytes, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(c->itw, itw.data(), tbytes, hipMemcpyHostToDevice) != hipSuccess ||
        (!tw2.empty() && (hipMemcpy(c->tw2, tw2.data(), tbytes, hipMemcpyHostToDevice) != hipSuccess ||
                          hipMemcpy(c->itw2, itw2.data(), tbytes, hipMemcpyHostToDevice) != hipSuccess)) ||
        hipDeviceSynchronize() != hipSuccess) {
        cg_destroy(c);
        return CG_EHIP;
    }
    bool ok = hipEventCreateWithFlags(&c->ev_fork, hipEventDisableTiming) == hipSuccess;
    ok = ok && side_acquire(c->device, c->side_default) && create_pair(c->side_own);
    for (int i = 0; i < 2 && ok; i++)
        ok = hipEventCreateWithFlags(&c->ev_join[i], hipEventDisableTiming) == hipSuccess;
    if (!ok) {
        cg_destroy(c);
        return CG_EHIP;
    }
    // one dry pass over every launch sequence fills the occupancy table
    c->dry = true;
    const int wrc = warm_launch_table(c);
    c->dry = false;
    if (wrc != CG_OK) {
        cg_destroy(c);
        return wrc;
    }
    *out = c;
    return CG_OK;
}

extern "C" int cg_destroy(cg_ctx *c)
{
    if (!c) return CG_OK;
    (void)hipDeviceSynchronize();
    if (c->ev_fork) (void)hipEventDestroy(c->ev_fork);
    for (int i = 0; i < 2; i++)
        if (c->ev_join[i]) (void)hipEventDestroy(c->ev_join[i]);
    destroy_pair(c->side_own);
    if (c->side_default[0]) side_release(c->device);
    if (c->dc) (void)hipFree(c->dc);
    if (c->tw) (void)hipFree(c->tw);
    if (c->itw) (void)hipFree(c->itw);
    if (c->tw2) (void)hipFree(c->tw2);
    if (c->itw2) (void)hipFree(c->itw2);
    if (c->tab) (void)hipFree(c->tab);
    for (uint32_t i = 0; i < 2 * c->prof_cap; i++) (void)hipEventDestroy(c->prof_ev[i]);
    delete[] c->prof_ev;
    delete[] c->prof_id;
    delete[] c->prof_bytes;
    delete[] c->prof_items;
    delete c->occ;
    delete c->occ_mu;
    delete c;
    return CG_OK;
}

static size_t limb_bytes(const cg_ctx *c) { return (size_t)c->N * 8; }

extern "C" int cg_get_sizes(const cg_ctx *c, cg_sizes *o)
{
    CG_REQUIRE(c && o);
    o->ct2_bytes = 2 * (size_t)c->k * limb_bytes(c);
    o->ct3_bytes = 3 * (size_t)c->k * limb_bytes(c);
    o->ksk_raw_bytes = (size_t)c->dnum * 2 * c->L * limb_bytes(c);
    o->ksk_bytes = o->ksk_raw_bytes;
    o->plain_bytes = (size_t)c->k * limb_bytes(c);
    o->ws_bytes_per_unit = (size_t)c->ws_total * limb_bytes(c);
    o->ct_ext_bytes = 2 * (size_t)c->KL * limb_bytes(c);
    return CG_OK;
}

extern "C" size_t cg_workspace_bytes(const cg_ctx *c, uint32_t batch)
{
    if (!c) return 0;
    return (size_t)c->ws_total * limb_bytes(c) * (batch ? batch : 1);
}

// Workspace carving: composite operations take their persistent buffers first and hand the
// rest to the primitive sequences, which start again from the pointer they are given.
struct Bump {
    char *p;
    size_t limb;
    template <class T> T *take(size_t limbs)
    {
        T *r = reinterpret_cast<T *>(p);
        p += limbs * limb;
        return r;
    }
};
static Bump bump(const cg_ctx *c, void *ws) { return Bump{static_cast<char *>(ws), limb_bytes(c)}; }

// ---------------------------------------------------------------------------
// launch helpers
// ---------------------------------------------------------------------------
// Transform kernels are persistent: the grid is at most the number of workgroups that are
// resident at once (what the runtime reports for this instantiation's registers and LDS), so
// that every workgroup starts immediately and walks over its rows with the next row prefetched.
template <auto KERNEL>
static unsigned ntt_grid(cg_ctx *c, size_t nwg, int threads)
{
    const void *key = reinterpret_cast<const void *>(KERNEL);
    int per_cu = 0;
    {
        std::lock_guard<std::mutex> g(*c->occ_mu);
        auto it = c->occ->find(key);
        if (it != c->occ->end()) per_cu = it->second;
    }
    if (per_cu == 0) {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, KERNEL, threads, 0) != hipSuccess || n < 1) n = 1;
        per_cu = n;
        std::lock_guard<std::mutex> g(*c->occ_mu);
        (*c->occ)[key] = per_cu;
    }
    const size_t resident = (size_t)per_cu * (size_t)c->n_cu;
    return (unsigned)(nwg < resident ? nwg : resident);
}
// What runs beside a product or a key switch: nothing (a call made alone, of whatever kind), or the other branches of a step; step_impl says which.
// crowd: their mod-ups have a row for every compute unit.  Beside such, rows are not taken in parts: these repeat a row's first stages on units
// that the others have work for.  us a step with whole rows / parts in the context's key switches, heads x ciphertexts: N = 8192,
// 6 x 7 (d2 = 128) 612 / 630, 10 x 6 694 / 726; N = 4096, 12 x 7 212 / 219; N = 16384, 4 x 3 586 / 607.
// longer: theirs is the chain with more dependent key switches, which the step waits for.
// wide: their summed rotations take ks_wide_kernel, a workgroup of which leaves no room on its compute unit.
// rows: of their mod-ups.  most: rotations of their largest round, where these count.
// leads: theirs is the chain with at least two dependent key switches fewer, and their (unit, prime) rows take one round.
struct Beside {
    bool others = false, crowd = false, wide = false, longer = false, leads = false;
    size_t rows = 0;
    uint32_t most = 0;
};

// elements per thread for this context's transforms
static int ntt_elems(const cg_ctx *c) { return c->elems; }

// Parts of a row in which a launch of `rows` rows is taken (ntt_fwd_part_kernel, ntt_inv_part_kernel), as a power of two: as many as
// have a compute unit each, four at most, two in an inverse transform at N = 8192 and none at N = 4096.  us a launch, whole rows / parts.
// Forward, N = 4096: 12 rows 6.0 / 5.5 (four), 100: 6.2 / 5.5 (two); N = 8192: 12 7.5 / 5.5, 64 7.8 / 5.6, 65 ... 128 rows 8.2 / 6.4 ... 8.4 / 6.9;
// N = 16384: 12 11.8 / 6.4, 64 12.6 / 8.2, 128 13.8 / 11.0.  Inverse, N = 4096: 12 rows 6.0 / 6.6, 100: 6.0 / 5.7 (two); N = 8192: 12 7.7 / 6.0 (four:
// 7.4), 64 8.1 / 6.5, 88 8.6 / 7.0, 128 8.7 / 7.6, 136 8.8 / 10.0; N = 16384: 12 13.5 / 10.1, 64 14.3 / 11.7 (four), 72 14.7 / 15.6.  At N = 8192 also where
// whole rows would take a second round for up to 3/8 of the compute units, and halves take one and a half: 260 rows 16.7 / 15.4, 340: 17.3 / 15.9,
// 384: 17.7 / 17.0, 448: 17.8 / 19.8.
static int row_parts(const cg_ctx *c, size_t rows, bool inverse)
{
    const size_t n = (size_t)c->n_cu;
    if (c->dry) return 0;
    if (inverse && c->logn == 13) return 2 * rows <= n || (rows > n && 8 * rows <= 11 * n) ? 1 : 0;
    if (inverse) return c->logn == 14 && 4 * rows <= n ? 2 : 0;
    return 4 * rows <= n ? 2 : 2 * rows <= n ? 1 : 0;
}
// The same for the accumulators of summed rotations: written a launch before they come from L2, where every part's own gather of them
// costs more than for callers' rows.  us a series, 7 rotations, N = 8192: 1 ciphertext (8 rows) 24.1 / 23.7, 4 (32) 27.0 / 26.8, 6 (48) 30.1 / 30.4,
// 8 (64) 31.5 / 33.3, 10 (80) 33.6 / 36.0, 12 (96) 35.8 / 37.5; 36 (288) 69.6 / 66.7, 41 (328) 75.9 / 73.8.  N = 16384: 1 (16) 40.2 / 38.8, 4 (64)
// 54.8 / 53.7; beside a step's other branches, which the work done twice holds up, 1 x 1 274 / 268, 3 x 1 361 / 361, 3 x 3 (48) 520 / 530, 4 x 1 (64)
// 377 / 384.
static int acc_parts(const cg_ctx *c, size_t rows, bool others)
{
    const size_t n = (size_t)c->n_cu;
    if (c->logn == 13 && !c->dry) return 8 * rows <= n || (rows > n && 8 * rows <= 11 * n) ? 1 : 0;
    return c->logn == 14 && !c->dry && (others ? 8 : 4) * rows <= n ? 2 : 0;
}
// two device ranges share at least one byte
static bool overlap(const void *a, size_t a_bytes, const void *b, size_t b_bytes)
{
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return x < y + b_bytes && y < x + a_bytes;
}
static bool overlap(const void *a, const void *b, size_t bytes) { return overlap(a, bytes, b, bytes); }
// The parts of a row read all of it, each in its own time: not where the results land on the rows that are read.
template <class LD, class ST> static bool apart(const LD &, const ST &, size_t) { return true; }
static bool apart(const LdRowsU64 &ld, const StU64 &st, size_t bytes) { return !overlap(ld.src, st.base, bytes); }
static bool apart(const LdInvU64 &ld, const StInvU64 &st, size_t bytes) { return !overlap(ld.src, st.dst, bytes); }
static bool apart(const LdInvF64 &ld, const StInvF64 &st, size_t bytes) { return !overlap(ld.src, st.dst, bytes); }
#define CG_PART(KERNEL, LG, LS, TW)                                                                            \
    return launch_kernel(KERNEL<LG, LS, LD, ST>, dim3((unsigned)nwg << LS), dim3(1u << (LG - LS - 3)), s, ld, st, \
                         (const double *)TW, (const DevConst *)c->dc, (int)nwg)

// parts: of a row (row_parts), where loader and storer allow them
template <class LD, class ST>
static int launch_fwd(cg_ctx *c, hipStream_t s, size_t nwg, LD ld, ST st, int kid, double bytes, int parts = 0)
{
    if (nwg == 0) return CG_OK;
    ProfScope ps(c, s, kid, bytes, (double)nwg);
    if constexpr (in_parts<LD, ST>::value) {
        switch (c->logn * 10 + (parts && apart(ld, st, nwg * limb_bytes(c)) ? parts : 0)) {
        case 121: CG_PART(ntt_fwd_part_kernel, 12, 1, c->tw);
        case 122: CG_PART(ntt_fwd_part_kernel, 12, 2, c->tw);
        case 131: CG_PART(ntt_fwd_part_kernel, 13, 1, c->tw);
        case 132: CG_PART(ntt_fwd_part_kernel, 13, 2, c->tw);
        case 141: CG_PART(ntt_fwd_part_kernel, 14, 1, c->tw);
        case 142: CG_PART(ntt_fwd_part_kernel, 14, 2, c->tw);
        default: break;
        }
    }
    // N = 8192: a launch with no more rows than compute units finishes a row sooner on 1024 threads
    const int e = (c->logn == 13 && !fwd_many<LD>::value && nwg <= (size_t)c->n_cu) ? c->elems : c->elems_fwd;
    const int threads = c->N / e;
#define CG_FWD(LG, EL)                                                                          \
    do {                                                                                        \
        const unsigned grid = ntt_grid<ntt_fwd_kernel<LG, EL, LD, ST>>(c, nwg, threads);        \
        if (c->dry) return CG_OK;                                                               \
        return launch_kernel(ntt_fwd_kernel<LG, EL, LD, ST>, dim3(grid), dim3(threads), s, ld, st, \
                             (const double *)c->tw, (const DevConst *)c->dc, (int)nwg);         \
    } while (0)
    switch (c->logn * 100 + e) {
    case 1416:
        if constexpr (ld_no_16384<LD>::value) return CG_EINVAL;
        else CG_FWD(14, 16);
    case 1208: CG_FWD(12, 8);
    case 1308:
        if constexpr (fwd_many<LD>::value) return CG_EINVAL;
        else CG_FWD(13, 8);
    case 1316: CG_FWD(13, 16);
    default: return CG_EINVAL;
    }
#undef CG_FWD
}
template <class LD, class ST>
static int launch_inv(cg_ctx *c, hipStream_t s, size_t nwg, LD ld, ST st, int kid, double bytes, int parts = 0)
{
    if (nwg == 0) return CG_OK;
    ProfScope ps(c, s, kid, bytes, (double)nwg);
    if constexpr (in_parts<LD, ST>::value) {
        switch (c->logn * 10 + (parts && apart(ld, st, nwg * limb_bytes(c)) ? parts : 0)) {
        case 131: CG_PART(ntt_inv_part_kernel, 13, 1, c->itw);
        case 142: CG_PART(ntt_inv_part_kernel, 14, 2, c->itw);
        default: break;
        }
    }
    // N = 8192, as forward: no more rows than compute units, and a row is done sooner on 1024 threads (product and
    // relinearisation: 1 unit 52.4 -> 48.6 us, 8 units 62.0 -> 58.5).  In a step, beside other branches, heads x ciphertexts: chains
    // 2 x 2 306 -> 298, 6 x 2 351 -> 337, 4 x 3 346 -> 332, 6 x 1 317 -> 320 (30 shapes of up to 12 products: -1.7 % on average); in rounds
    // 8 x 1 211 -> 206, 4 x 3 229 -> 223, 5 x 1 189 -> 194, with a transformed cache 4 x 3 219 -> 228, 11 x 1 250 -> 246 (60: no difference).
    const int e = (c->logn == 13 && inv_wide<LD>::value && 2 * nwg > (size_t)inv_wide<LD>::value * c->n_cu) ? 16 : ntt_elems(c);
    const int threads = c->N / e;
#define CG_INV(LG, EL)                                                                          \
    do {                                                                                        \
        const unsigned grid = ntt_grid<ntt_inv_kernel<LG, EL, LD, ST>>(c, nwg, threads);        \
        if (c->dry) return CG_OK;                                                               \
        return launch_kernel(ntt_inv_kernel<LG, EL, LD, ST>, dim3(grid), dim3(threads), s, ld, st, \
                             (const double *)c->itw, (const DevConst *)c->dc, (int)nwg);        \
    } while (0)
    switch (c->logn * 100 + e) {
    case 1416:
        if constexpr (ld_no_16384<LD>::value) return CG_EINVAL;
        else CG_INV(14, 16);
    case 1208: CG_INV(12, 8);
    case 1308: CG_INV(13, 8);
    case 1316:
        if constexpr (inv_wide<LD>::value) CG_INV(13, 16);
        else return CG_EINVAL;
    default: return CG_EINVAL;
    }
#undef CG_INV
}
// ct x pt of every row of densely packed ciphertexts with plaintext (unit * pstride + pofs).  A whole
// row per 1024 threads also at N = 8192: the two transforms of a row follow each other without a trip
// to memory that a second workgroup on the unit could cover.
template <class ST>
static int launch_mulplain(cg_ctx *c, hipStream_t s, size_t nwg, const uint64_t *src, const double *plain, int pstride,
                           int pofs, ST st, double bytes)
{
    ProfScope ps(c, s, KID_MULPLAIN, bytes, (double)nwg);
#define CG_MP(LG, EL)                                                                                        \
    do {                                                                                                     \
        const unsigned threads = (1u << LG) / EL;                                                            \
        const unsigned grid = ntt_grid<ntt_mulplain_kernel<LG, EL, ST>>(c, nwg, (int)threads);               \
        if (c->dry) return CG_OK;                                                                            \
        return launch_kernel(ntt_mulplain_kernel<LG, EL, ST>, dim3(grid), dim3(threads), s, src, plain,      \
                             pstride, pofs, st, (const double *)c->tw, (const double *)c->itw,               \
                             (const DevConst *)c->dc, (int)nwg);                                             \
    } while (0)
    switch (c->logn) {
    case 12: CG_MP(12, 8);
    case 13: CG_MP(13, 8);
    case 14: CG_MP(14, 16);
    default: return CG_EINVAL;
    }
#undef CG_MP
}
static unsigned pw_blocks(const cg_ctx *c, size_t rows) { return (unsigned)((rows * c->N + PW_THREADS - 1) / PW_THREADS); }
#define CG_TRY(expr) do { int rc_ = (expr); if (rc_ != CG_OK) return rc_; } while (0)

// ---------------------------------------------------------------------------
// internal operations (arguments already validated)
// ---------------------------------------------------------------------------
// one pointwise launch, bracketed by the timing scope
#define CG_LAUNCH_PW(kid, bytes, items, kernel, blocks, ...)                                                \
    do {                                                                                               \
        if (c->dry) break;                                                                             \
        int rc_pw_;                                                                                    \
        {                                                                                              \
            ProfScope ps_(c, s, kid, bytes, items);                                                    \
            rc_pw_ = launch_kernel(kernel, dim3(blocks), dim3(PW_THREADS), s, __VA_ARGS__);            \
        }                                                                                              \
        CG_TRY(rc_pw_);                                                                                \
    } while (0)

// Summed inner products whose words are asked for a rotation ahead: with one or two ciphertexts a thread, where there are registers for two rotations' and few
// waves to cover a wait, and at N = 8192, from more than one workgroup per compute unit on, only while the keys of a prime leave an eighth of an XCD's L2 (4 MB)
// to the digits: fewer waves fit on a unit then, and beyond L2 they no longer share what they read.  us a series with mod-up and mod-down, words
// asked for as they are multiplied / ahead.  N = 8192, three digits (0.375 MB a rotation): 1 ciphertext, 7 rotations 22.4 / 21.4, 15 28.1 / 24.7; 2, 15 29.2 / 27.3; 6, 7 29.3 / 28.9,
// 9 30.9 / 30.0; 12, 7 35.7 / 35.6; 16, 7 39.1 / 39.1; 14, 9 41.3 / 42.1; with more keys 6, 15 36.3 / 38.8; 8, 11 36.2 / 36.7; 10, 15 46.3 / 52.7; 12, 15 46.1 / 47.5; 18, 11 50.4 / 52.1;
// two digits, 12, 15 (3.75 MB) 38.6 / 36.4, 31 54.5 / 60.4; four, 12, 7 43.6 / 44.7; six, one a thread, 4, 7 45.3 / 46.8, two, 12, 7 81.7 / 76.8, 15 139 / 124.  N = 4096, two digits, 4, 15
// 23.2 / 20.6, 24, 31 53.1 / 47.6; N = 16384, three, 6, 15 95.5 / 92.8.  (With four and eight a thread no difference and up to +12 %.)
static bool sum_keys_stay(const cg_ctx *c, size_t blocks, uint32_t n_rot, bool others)
{
    const size_t keys = 2 * (size_t)c->dnum * n_rot * limb_bytes(c);      // of one prime
    return c->logn != 13 || c->dnum == 1 || 2 * keys < (7u << 20) || 2 * blocks <= (others ? 3 : 2) * (size_t)c->n_cu;
}
static bool ks_sum_ahead_wins(const cg_ctx *c, uint32_t u, size_t blocks, uint32_t n_rot, bool others)
{
    return u <= 2 && n_rot > 1 && (sum_keys_stay(c, blocks, n_rot, others) || (c->dnum > 4 && u == 2));
}
// Summed inner products of a series of rotations.  Ciphertexts per thread: as many as leave every
// compute unit three workgroups and no more than a quarter of the last group's places empty.  us a series with mod-up and mod-down at
// one / two / four / eight a thread, 7 rotations, N = 8192: 12 ciphertexts 39.4 / 36.4 / 38.1 / 40.6, 24: 58.2 / 52.1 / 49.8 / 53.5, 36: 76.6 / 67.1 / 66.4 / 70.4,
// 40: 80.7 / 70.3 / 67.7 / 73.5; N = 4096, 24: 28.5 / 28.0 / 28.7 / 30.9, 42: 34.3 / 32.2 / 34.8 / 36.1; N = 16384, 4: 62.1 / 52.3 / 49.1 / 54.2, 12: 145 / 116 / 106 / 108.
// 3 rotations, N = 8192: 20 37.6 / 35.4 / 36.4 / 38.5, 24 45.2 / 42.8 / 42.6 / 45.3, 32: 50.1 / 46.6 / 46.5 / 47.6, 40: 60.4 / 56.2 / 55.8 / 59.8, but 28 47.3 / 44.7 / 45.0 / 46.0, 36 57.8 / 54.1 /
// 55.0 / 57.6 and 41 61.8 / 57.6 / 58.3 / 59.4, where two would be better than the rule's four.
template <int DNUM>
static int launch_ks_sum_d(cg_ctx *c, hipStream_t s, const uint64_t *dig, const HoistTab &T, uint32_t n_rot, double *acc,
                           uint32_t batch, bool others)
{
    const size_t per = (size_t)c->L * c->N / PW_THREADS;
    uint32_t u = 8;
    auto groups = [&]() { return (batch + u - 1) / u; };
    while (u > 1 && (per * groups() < 3 * (size_t)c->n_cu || 4 * (size_t)groups() * u > 5 * (size_t)batch)) u /= 2;
    const dim3 block(PW_THREADS), grid((unsigned)(per * groups()));
    const DevConst *dc = c->dc;
    const bool ahead = ks_sum_ahead_wins(c, u, per * groups(), n_rot, others);
#define CG_KSSUM(U, AHEAD) return launch_kernel(ks_sum_kernel<DNUM, U, AHEAD>, grid, block, s, dig, T, (int)n_rot, acc, (int)batch, dc)
    switch (u) {
    case 8: CG_KSSUM(8, false);
    case 4: CG_KSSUM(4, false);
    case 2: if (ahead) CG_KSSUM(2, true); CG_KSSUM(2, false);
    default: if (ahead) CG_KSSUM(1, true); CG_KSSUM(1, false);
    }
#undef CG_KSSUM
}
static int launch_ks_sum(cg_ctx *c, hipStream_t s, double bytes, const uint64_t *dig, const HoistTab &T, uint32_t n_rot,
                         double *acc, uint32_t batch, bool others)
{
    if (c->dry) return CG_OK;
    ProfScope ps(c, s, KID_KSSUM, bytes, (double)batch);
    switch (c->dnum) {
    case 1: return launch_ks_sum_d<1>(c, s, dig, T, n_rot, acc, batch, others);
    case 2: return launch_ks_sum_d<2>(c, s, dig, T, n_rot, acc, batch, others);
    case 3: return launch_ks_sum_d<3>(c, s, dig, T, n_rot, acc, batch, others);
    case 4: return launch_ks_sum_d<4>(c, s, dig, T, n_rot, acc, batch, others);
    case 5: return launch_ks_sum_d<5>(c, s, dig, T, n_rot, acc, batch, others);
    default: return launch_ks_sum_d<6>(c, s, dig, T, n_rot, acc, batch, others);
    }
}

// one ciphertext a thread, and the rows of the mod-down before
static int launch_ks_sum_after(cg_ctx *c, hipStream_t s, double bytes, const uint64_t *dig, const HoistTab &T, uint32_t n_rot, double *acc, uint32_t batch,
                               const ModdownArgs &A, const ModdownHoist &H)
{
    ProfScope ps(c, s, KID_KSSUM, bytes, (double)batch);
    const unsigned sums = (unsigned)((size_t)batch * c->L * c->N / PW_THREADS), down = (unsigned)((size_t)batch * 2 * c->k * c->N / (2 * PW_THREADS));
    const DevConst *dc = c->dc;
#define CG_KSAFTER(D) return launch_kernel(ks_sum_after_kernel<D>, dim3(sums + down), dim3(PW_THREADS), s, dig, T, (int)n_rot, acc, (int)batch, (int)sums, A, H, dc)
    switch (c->dnum) {
    case 1: CG_KSAFTER(1);
    case 2: CG_KSAFTER(2);
    case 3: CG_KSAFTER(3);
    default: return CG_EINVAL;
    }
#undef CG_KSAFTER
}

// The kernels that take a (unit, prime) through several transforms in one workgroup work in rounds of one row per compute
// unit, and a round takes as long for one row as for all of them; the launches of single transforms that they replace
// spread over the chip in finer pieces.  Taken while no more units than this stay idle in the last round, in 256ths
// of the compute units, with one, two and three rounds; from the fourth round on it does not matter.
struct IdleLimits {
    int one, two, three;
};
static bool rounds_pay(const cg_ctx *c, size_t rows, IdleLimits lim)
{
    const size_t n = (size_t)c->n_cu, rounds = (rows + n - 1) / n, idle = rounds * n - rows;
    return rounds > 3 || 256 * idle <= n * (size_t)(rounds == 1 ? lim.one : rounds == 2 ? lim.two : lim.three);
}

// Two units to a workgroup of ks_sum_row_kernel at N = 8192, where a round of pairs takes the time of 1.84 rounds of one and there are
// few enough of them.  us, one unit / two, three digits, 7 rotations: 64 ciphertexts (one round / one) 82 / 117, 107 (two / one)
// 152 / 139, 128: 163 / 151, 192 (three / two) 242 / 267, 193 (four / two) 286 / 266, 320 (five / three) 400 / 412, 321 (six / three) 438 / 410, 768: 932 / 880;
// 3 rotations, 128: 129 / 120, 192: 191 / 211, 384: 378 / 354; two digits, 7 rotations, 128: 104 / 98, 256 (three / two) 187 / 204; six, 111: 489 / 431.  At N = 4096,
// where a compute unit holds two workgroups of one unit, pairs gain nothing: two digits, 7 rotations, 256: 88 / 95, 512: 150 / 150, 1536: 462 / 463 (before sums were
// added up unreduced with one unit, which 256 now takes in 83).
static bool ks_sum_pairs(const cg_ctx *c, uint32_t batch)
{
    if (c->logn != 13) return false;
    const size_t n = (size_t)c->n_cu, one = ((size_t)batch * c->L + n - 1) / n;
    const size_t two = ((size_t)((batch + 1) / 2) * c->L + n - 1) / n;
    return 184 * two < 100 * one;
}
// mod-up, summed inner products and inverse transforms in one launch, modulo the primes from r0 on
static int launch_ks_sum_row(cg_ctx *c, hipStream_t s, const uint64_t *src, size_t src_stride, const HoistTab &T,
                             uint32_t n_rot, double *acc, uint32_t batch, int r0 = 0)
{
    const int primes = c->L - r0;
    const double bytes = (double)limb_bytes(c) * ((c->k + 2.0 * primes) * batch + 2.0 * c->dnum * primes * n_rot);
    ProfScope ps(c, s, KID_KSSUMROW, bytes, (double)batch * primes);
    const bool pairs = ks_sum_pairs(c, batch);
#define CG_KSSUMROW(LG, U)                                                                                    \
    do {                                                                                                      \
        const size_t nwg = (size_t)((batch + U - 1) / U) * primes;                                            \
        const unsigned threads = (1u << LG) / 8;                                                              \
        const unsigned grid = ntt_grid<ks_sum_row_kernel<LG, 8, U>>(c, (nwg + 7) / 8 * 8, (int)threads);      \
        if (c->dry) break;                                                                                    \
        return launch_kernel(ks_sum_row_kernel<LG, 8, U>, dim3(grid), dim3(threads), s,                       \
                             LdModup<false, 1>{src, src_stride, 0, c->logn}, T, (int)n_rot, (int)batch,       \
                             StInvF64{acc, c->logn}, (const double *)c->tw, (const double *)c->itw,           \
                             (const DevConst *)c->dc, (int)nwg, r0);                                          \
    } while (0)
    switch (c->logn) {
    case 12:
        CG_KSSUMROW(12, 1);
        return CG_OK;
    case 13:
        if (pairs || c->dry) CG_KSSUMROW(13, 2);
        if (!pairs) CG_KSSUMROW(13, 1);
        return CG_OK;
    default: return CG_EINVAL;
    }
#undef CG_KSSUMROW
}
// the same modulo the ciphertext primes, with the mod-down
static int launch_ks_sum_down(cg_ctx *c, hipStream_t s, const uint64_t *src, size_t src_stride, const HoistTab &T, const ModdownArgs &A,
                              const ModdownHoist &H)
{
    const double bytes = (double)limb_bytes(c) * ((7.0 * c->k + 2.0) * A.batch + 2.0 * c->dnum * c->k * H.n_sum);
    ProfScope ps(c, s, KID_KSSUMDOWN, bytes, (double)A.batch * c->k);
    const size_t nwg = (size_t)(A.batch + 1) / 2 * c->k;
    const unsigned grid = ntt_grid<ks_sum_down_kernel<13, 8>>(c, (nwg + 7) / 8 * 8, 1024);
    if (c->dry) return CG_OK;
    return launch_kernel(ks_sum_down_kernel<13, 8>, dim3(grid), dim3(1024), s, LdModup<false, 1>{src, src_stride, 0, c->logn}, T, A, H,
                         (const double *)c->tw, (const double *)c->itw, (const DevConst *)c->dc, (int)nwg);
}
// Pairs of units: the accumulators modulo the special prime in a launch of their own, those of the ciphertext primes with the mod-down behind them in
// the kernel, where the two launches take no more rounds of workgroups together than the one (their last rounds are both partly empty), or, with
// up to three digits and eight rotations, from four units per compute unit on, where a round more costs less than the mod-down's way through
// memory.  us, one launch and mod-down / two, 7 rotations, three digits: 460 ciphertexts 557 / 487, 512 584 / 510, 900 1095 / 972, 1024 1153 / 1046, 1536 1723 / 1568; a round
// more: 256 296 / 348, 384 441 / 472, 600 703 / 714, 640 728 / 719, 1100 1266 / 1219, 1280 1434 / 1361 and with 15 rotations 1100 1816 / 1840; four digits, 400 681 / 730,
// 512 863 / 776, 640 1143 / 1032; six, 500 1635 / 1500.
static bool ks_sum_down_wins(const cg_ctx *c, uint32_t batch, uint32_t n_rot)
{
    if (c->logn != 13 || c->nsp != 1 || c->alpha != 1) return false;
    if (c->dry) return c->dry_rows;
    if (!ks_sum_pairs(c, batch)) return false;
    const size_t n = (size_t)c->n_cu, sets = (batch + 1) / 2;
    auto rounds = [&](size_t primes) { return (sets * primes + n - 1) / n; };
    return rounds(1) + rounds(c->k) <= rounds(c->L) || (c->dnum <= 3 && n_rot <= 8 && batch >= 4 * n);
}
// us with the mod-down and other keys on every call, launches of single transforms / one.  N = 8192, three digits, 7 rotations: 32 ciphertexts (128 units idle) 56.5 / 63.9,
// 36 (112) 67.5 / 65.7, 40 (96): 68.7 / 66.4, 42 (88): 73.9 / 66.7, 64: 102 / 79; 3 rotations, 32: 47.7 / 50.3, 36: 55.9 / 51.8, 42: 60.7 / 53.3;
// 15 rotations, 36 92 / 96, 42: 101 / 97, 48 (64): 114 / 101.  At N = 4096 a unit holds two workgroups.  Two digits, 7 rotations, 42 (130 idle): 32.2 / 33.4, 43 (127): 36.2 / 33.4,
// 86 (254): 49.9 / 47.8, 107 (191): 54.9 / 50.1.  Three digits, 7 rotations: 33 (124 idle) 41.0 / 41.5, 42 (88): 44.2 / 41.6, 72 (224):
// 62.1 / 62.3, 84 (176): 66.6 / 62.6, 90 (152): 71.9 / 65.0; six digits: 20 (116) 61.1 / 66.5, 24 (88): 68.4 / 68.5, 26 (74): 78.3 / 68.8.
// The limits at N = 8192 are older than these figures, which would have them at 3/7 of the units in one round and 3/4 and more in the second and third: 7 rotations, 65
// (252 idle) 119 / 118, 80 (192): 131 / 122, 96 (128): 153 / 131, 103 (100): 170 / 136, 129 (252) 215 / 212, 150 (168): 241 / 220, 166 (104): 259 / 227; 3 rotations, 80:
// 105 / 94, 150: 193 / 173; two digits, 7 rotations, 110 (182): 103 / 95, 136 (104): 132 / 103, and in one round 43 (127) 57.6 / 53.0, 48 (112): 58.4 / 51.8.
// Pairs of units (ks_sum_pairs), four digits and more: from a quarter more rows than compute units on.  N = 8192, 7 rotations: four
// digits, 63 ciphertexts (315 rows) 200 / 154, 81 (405): 278 / 168; six, 37 (259): 202 / 208, 45 (315): 239 / 215, 54: 275 / 222.
static bool ks_sum_row_wins(const cg_ctx *c, uint32_t batch)
{
    if (c->logn > 13 || c->alpha != 1) return false;
    if (c->dry) return c->dry_rows;
    if (c->dnum > 3 && ks_sum_pairs(c, batch) && 4 * (size_t)batch * c->L >= 5 * (size_t)c->n_cu) return true;
    return rounds_pay(c, (size_t)batch * c->L, c->logn == 13 ? IdleLimits{89, 102, 102}
                                             : c->dnum <= 2 ? IdleLimits{128, 256, 256} : IdleLimits{84, 176, 256});
}

// the same at N = 16384; a relinearisation is the series of one rotation by g = 1
static int launch_ks_wide(cg_ctx *c, hipStream_t s, const uint64_t *src, size_t src_stride, const HoistTab &T, uint32_t n_rot,
                          double *acc, uint32_t batch)
{
    const double bytes = (double)limb_bytes(c) * ((c->k + 2.0 * c->L) * batch + 2.0 * c->dnum * c->L * n_rot);
    ProfScope ps(c, s, KID_KSSUMROW, bytes, (double)batch * c->L);
    const size_t nwg = (size_t)batch * c->L;
#define CG_KSWIDE(A)                                                                                          \
    do {                                                                                                      \
        const unsigned grid = ntt_grid<ks_wide_kernel<A>>(c, (nwg + 7) / 8 * 8, 1024);                        \
        if (c->dry) return CG_OK;                                                                             \
        return launch_kernel(ks_wide_kernel<A>, dim3(grid), dim3(1024), s, LdModup<false, A>{src, src_stride, 0, c->logn}, T, \
                             (int)n_rot, (int)batch, StInvF64{acc, c->logn}, (const double *)c->tw, (const double *)c->itw, \
                             (const DevConst *)c->dc, (int)nwg);                                              \
    } while (0)
    if (c->alpha == 1) CG_KSWIDE(1);
    CG_KSWIDE(2);
#undef CG_KSWIDE
}
// us with the mod-down, N = 16384, six primes, two special ones, three launches / one; 1, 3 and 7 rotations: 16 units (128 compute units
// idle) 88 / 99, 101 / 122, 126 / 165, 20 (96): 108 / 108, 126 / 130, 160 / 172, 21 (88): 111 / 109, 130 / 131, 164 / 175, 22 (80): 128 / 113, 146 / 135,
// 181 / 178, 26 (48): 136 / 119, 158 / 141, 210 / 184, relinearisations of 21 and 22 101 / 101, 113 / 102; 36 (224): 197 / 197,
// 227 / 230, 286 / 299, 40 (192): 210 / 203, 238 / 237, 300 / 309, 44 (160): 238 / 209, 268 / 242, 343 / 319, 64: 321 / 268, 369 / 309,
// 473 / 394; 80 (128): 416 / 361, 468 / 417, 595 / 535.
// Alone, contexts of 16 heads in rounds, 1, 2, 3 ciphertexts: 630 / 715, 698 / 791, 770 / 861; scores of 18 products 589 / 621.
// In a step, us of the whole step, heads x ciphertexts; six primes unless said.  The scores' summed rotations of one round pay a little sooner: 10 x 2
// (96 idle) 977 / 942, 7 x 3 (88) 872 / 859, 5 x 4 833 / 837, 2 x 10 772 / 784, four primes 9 x 3 (94) 745 / 730; at 104 and 112 idle as many lose (3 x 6 733 / 755,
// 6 x 3 815 / 830, 18 x 1 1165 / 1180) as gain (9 x 2 871 / 846).  The context's sooner still where the scores' take whole units already (wide): 16 x 2 (128
// idle) 1409 / 1381, with a transformed cache 1419 / 1400, 16 x 3 1853 / 1768, 16 x 4 2273 / 2218, 17 x 5 (120) 2945 / 2813, 18 x 3 (112) 2056 / 2027; mixed above: 15 x 2 (136)
// 1365 / 1333, with a transformed cache 1382 / 1408, 15 x 4 2085 / 2055, 2009 / 2021, 14 x 2 (144) 1289 / 1291, 1289 / 1329.  Where they do not, never: 16 x 1 1015 / 1085, 17 x 1 1113 / 1152,
// four primes 22 x 2 1202 / 1250, 23 x 2 1260 / 1280, two 43 x 2 1172 / 1202, 47 x 2 1249 / 1286.  Relinearisations only
// from the second round on (14 x 2, 32 idle, 1269 / 1300, 16 x 2 1372 / 1411; 16 x 3, 128 in the second, 1797 / 1766, 16 x 4 2279 / 2205); two rounds no sooner than
// at 144 idle (11 x 4, 160 idle, 1675 / 1684, 10 x 4 1506 / 1555).
static bool ks_wide_wins(const cg_ctx *c, uint32_t batch, bool relin, Beside beside)
{
    if (c->logn != 14) return false;
    if (c->dry) return c->dry_rows;
    const size_t rows = (size_t)batch * c->L;
    if (relin && beside.others && rows <= (size_t)c->n_cu) return false;
    return rounds_pay(c, rows, IdleLimits{beside.wide ? 128 : beside.others ? 96 : 80, 144, 160});
}

// whole key switches, summed rotations or not, in one launch
template <int MODE>
static int launch_ks_unit(cg_ctx *c, hipStream_t s, const uint64_t *src, size_t src_stride, uint32_t galois,
                          const HoistTab &T, const ModdownArgs &A, const ModdownHoist &H, double *scratch, double add_rows)
{
    const double bytes = (double)limb_bytes(c) * ((3.0 * c->k + add_rows) * A.batch +
                                                  2.0 * c->dnum * c->L * (MODE == KS_SUM ? H.n_sum : 1));
    ProfScope ps(c, s, KID_KSUNIT, bytes, (double)A.batch);
#define CG_KSUNIT(LG)                                                                                         \
    do {                                                                                                     \
        const unsigned threads = (1u << LG) / 8;                                                             \
        const unsigned grid = ntt_grid<ks_unit_kernel<LG, 8, MODE>>(c, (size_t)A.batch, (int)threads);       \
        if (c->dry) return CG_OK;                                                                            \
        return launch_kernel(ks_unit_kernel<LG, 8, MODE>, dim3(grid), dim3(threads), s,                      \
                             LdModup<MODE == KS_ROTATE, 1>{src, src_stride, galois, c->logn}, T, A, H, scratch, \
                             (const double *)c->tw, (const double *)c->itw, (const DevConst *)c->dc);        \
    } while (0)
    switch (c->logn) {
    case 12: CG_KSUNIT(12);
    case 13: CG_KSUNIT(13);
    default: return CG_EINVAL;
    }
#undef CG_KSUNIT
}
// Whole units are coarse pieces: taken where the last round of workgroups leaves a tenth of the compute units idle at
// most, from two workgroups per unit on at N = 4096, and where the keys of a prime stay in an XCD's L2, whose
// workgroups are at different primes.  us by row / by unit with another key on every call.  N = 8192, three digits, rotations:
// 231 units 181 / 182, 256: 188 / 187, 300: 234 / 344, 450: 372 / 353, 600: 474 / 515, 693: 529 / 525, 768: 580 / 537; 3 summed rotations, 231: 226 / 213, 256: 237 / 220,
// 693 668 / 611, 768: 700 / 633, but with the mod-down in the kernel that sums (ks_sum_down_wins) 461: 369 / 406, 512 389 / 425, which the rule does not look at; two digits, rotations, 231: 114 / 106, 420: 191 / 204, 461: 218 / 208.  N = 4096, two digits, relinearisation: 420 units 86 / 79,
// 461: 99 / 84, 768: 154 / 128; rotation, 256: 55 / 67, 461: 106 / 91; 7 summed rotations, 256: 83 / 93, 461: 159 / 144.
// Relinearisations of three digits at N = 8192 go by unit in the second round, and from the third on with a sixteenth idle at most.  That line is older than the
// kernel, which has since transformed both sums back together and gains wherever the rule for the others holds: 231 units 163 / 151,
// 256: 171 / 160, 420 (which that leaves out) 313 / 292, 461: 353 / 298, 512: 372 / 311, 693: 501 / 439, 720: 532 / 446, 768: 553 / 459; two digits, 231: 104 / 93, 461: 215 / 184.
static bool ks_unit_wins(const cg_ctx *c, size_t batch, size_t n_rot, bool relin = false)
{
    if (c->logn > 13 || c->alpha != 1 || c->nsp != 1) return false;
    if (c->dry) return c->dry_units;
    const size_t n = (size_t)c->n_cu, rounds = (batch + n - 1) / n;
    if (relin && c->logn == 13 && c->dnum > 2 && (rounds == 1 || (rounds > 2 && 16 * batch < 15 * rounds * n))) return false;
    return 10 * batch >= 9 * rounds * n && (c->logn == 13 || rounds > 1) &&
           2 * c->dnum * n_rot * limb_bytes(c) <= (size_t)2 << 20;
}

// mod-down of a summed series of rotations, one output row per workgroup
static int launch_moddown_sum(cg_ctx *c, hipStream_t s, double bytes, size_t batch, const ModdownArgs &A,
                              const ModdownHoist &H)
{
    if (c->dry) return CG_OK;
    ProfScope ps(c, s, KID_MODDOWN_SUM, bytes, (double)batch);
    const dim3 block(1024);
    const size_t rows = batch * 2 * c->k;
    const DevConst *dc = c->dc;
#define CG_MDS(LG, SP) \
    return launch_kernel(moddown_sum_kernel<LG, SP>, dim3((unsigned)(rows * moddown_sum_split<LG>())), block, s, A, H, dc)
    switch (c->logn * 10 + c->nsp) {
    case 121: CG_MDS(12, 1);
    case 122: CG_MDS(12, 2);
    case 131: CG_MDS(13, 1);
    case 132: CG_MDS(13, 2);
    case 141: CG_MDS(14, 1);
    case 142: CG_MDS(14, 2);
    default: return CG_EINVAL;
    }
#undef CG_MDS
}
// mod-down per pair of coefficients; hoisted: the units are the rotations of a series
template <bool HOIST>
static int launch_moddown(cg_ctx *c, hipStream_t s, double bytes, size_t units, const ModdownArgs &A,
                          const ModdownHoist &H)
{
    if (c->dry) return CG_OK;
    ProfScope ps(c, s, KID_MODDOWN, bytes, (double)units);
    const dim3 grid(pw_blocks(c, units * 2) / 2), block(PW_THREADS);
    const DevConst *dc = c->dc;
    return c->nsp == 1 ? launch_kernel(moddown_kernel<HOIST, 1>, grid, block, s, A, H, dc)
                       : launch_kernel(moddown_kernel<HOIST, 2>, grid, block, s, A, H, dc);
}

// N = 16384: operands lifted to all k + l primes, first transform stage taken, in half rows
static int launch_lift(cg_ctx *c, hipStream_t s, const MulSrc &src, size_t polys, double *dst)
{
    const double bytes = (double)limb_bytes(c) * polys * (c->k + c->KL);
    const unsigned blocks = (unsigned)(polys * (size_t)(c->N / 2 / PW_THREADS));
#define CG_LIFT(K) CG_LAUNCH_PW(KID_LIFT, bytes, (double)polys, lift_kernel<K>, blocks, src, dst, c->dc)
    switch (c->k) {
    case 1: CG_LIFT(1); break;
    case 2: CG_LIFT(2); break;
    case 3: CG_LIFT(3); break;
    case 4: CG_LIFT(4); break;
    case 5: CG_LIFT(5); break;
    default: CG_LIFT(6); break;
    }
#undef CG_LIFT
    return CG_OK;
}
// the half rows of lifted operands transformed in place; up to one per compute unit on 1024 threads (launch_fwd)
static int launch_fwd_half(cg_ctx *c, hipStream_t s, const MulSrc &src, size_t polys, double *dst)
{
    const size_t nwg = polys * 2 * c->KL;
    ProfScope ps(c, s, KID_FWD_HALF, (double)limb_bytes(c) * nwg, (double)nwg);
#define CG_HALF(EL)                                                                                            \
    do {                                                                                                      \
        const unsigned threads = 8192 / EL, grid = ntt_grid<ntt_fwd_kernel<13, EL, LdHalf, StF64>>(c, nwg, (int)threads); \
        if (c->dry) return CG_OK;                                                                             \
        return launch_kernel(ntt_fwd_kernel<13, EL, LdHalf, StF64>, dim3(grid), dim3(threads), s,             \
                             LdHalf{dst, src}, StF64{dst, 13}, (const double *)c->tw2, (const DevConst *)c->dc, (int)nwg); \
    } while (0)
    if (nwg <= (size_t)c->n_cu) CG_HALF(8);
    CG_HALF(16);
#undef CG_HALF
}
// Every polynomial named by src -> its transform over the k ciphertext primes and the l auxiliary
// primes (centred lift), rows dst[poly][k+l][N], lazy.
static int transform_ext(cg_ctx *c, hipStream_t s, const MulSrc &src, size_t polys, double *dst)
{
    if (c->logn == 14) {
        CG_TRY(launch_lift(c, s, src, polys, dst));
        return launch_fwd_half(c, s, src, polys, dst);
    }
    const double LB = (double)limb_bytes(c);
    const double in_rows = (double)polys * c->k;
    const StF64 st{dst, c->logn};
    // Both kinds of rows in one launch while they are at most two per compute unit: product and relinearisation, us in two launches / one: N = 8192, one product 55 / 46, 8: 65 / 57, 16:
    // 83 / 79, 18 (504 rows) 92 / 82; N = 4096, 1: 36 / 30, 16: 45.6 / 43.3, 25 (500) 54 / 48.  Large launches are faster apart (the lifts' code for the plain rows).
    if (polys * c->KL <= (size_t)c->n_cu * 2) {
        const double bytes = LB * (in_rows + (double)polys * c->KL);
        switch (c->k) {
        case 1: return launch_fwd(c, s, polys * c->KL, LdMulExt<1>{src}, st, KID_FWD_MULEXT, bytes);
        case 2: return launch_fwd(c, s, polys * c->KL, LdMulExt<2>{src}, st, KID_FWD_MULEXT, bytes);
        case 3: return launch_fwd(c, s, polys * c->KL, LdMulExt<3>{src}, st, KID_FWD_MULEXT, bytes);
        case 4: return launch_fwd(c, s, polys * c->KL, LdMulExt<4>{src}, st, KID_FWD_MULEXT, bytes);
        case 5: return launch_fwd(c, s, polys * c->KL, LdMulExt<5>{src}, st, KID_FWD_MULEXT, bytes);
        default: return launch_fwd(c, s, polys * c->KL, LdMulExt<6>{src}, st, KID_FWD_MULEXT, bytes);
        }
    }
    CG_TRY(launch_fwd(c, s, polys * c->k, LdMulQ{src}, st, KID_FWD_MULQ, LB * 2.0 * in_rows));
    const double aux_bytes = LB * (in_rows + (double)polys * c->l);
    switch (c->k) {
    case 1: return launch_fwd(c, s, polys * c->l, LdMulAux<1>{src}, st, KID_FWD_MULB, aux_bytes);
    case 2: return launch_fwd(c, s, polys * c->l, LdMulAux<2>{src}, st, KID_FWD_MULB, aux_bytes);
    case 3: return launch_fwd(c, s, polys * c->l, LdMulAux<3>{src}, st, KID_FWD_MULB, aux_bytes);
    case 4: return launch_fwd(c, s, polys * c->l, LdMulAux<4>{src}, st, KID_FWD_MULB, aux_bytes);
    case 5: return launch_fwd(c, s, polys * c->l, LdMulAux<5>{src}, st, KID_FWD_MULB, aux_bytes);
    default: return launch_fwd(c, s, polys * c->l, LdMulAux<6>{src}, st, KID_FWD_MULB, aux_bytes);
    }
}

// mul_row_kernel; cached: in an attention call, where it pays with more units idle, beside other branches and alone.  us of a product with its scaling, three
// launches / one.  N = 8192, three primes: 18 products (130 units idle) 55.2 / 57.3, 19 (123): 65.8 / 57.6, 42 (218): 103 / 109, 55 (127): 130 / 114; two: 25 (131)
// 50.5 / 51.5, 26 (126): 60.7 / 51.4.  N = 4096, three primes: 16 (144) 32.2 / 34.6, 20 (116): 37.8 / 36.4, 23 (95): 40.1 / 36.3, 42 (218): 54.5 / 55.3, 49 (169): 66.5 / 57.6;
// two: 16 (176) 26.7 / 29.2, 24 (136): 29.6 / 31.9, 26 (126): 35.5 / 32.9, 52 (252): 50.8 / 46.9, 58 (222): 51.6 / 50.7, 68 (172): 58.2 / 52.2.  48 products over a cache (176 idle in
// the second round): chain step of 12 heads 686 / 656, scores alone 307 / 294; 49 (169) 340 / 315, 44 (204) 295 / 294.  The second round's limit for other products, and
// the first one's with three primes at N = 4096, are older than these figures and could lie where the cache's does: N = 8192, 44 products (204) 109 / 110, 48 (176): 113 / 111, 50 (162):
// 126 / 112, 52 (148): 128 / 112; two primes, 60 (212) 95.7 / 95.9, 70 (162): 119 / 98.  A row of 16384 leaves no registers for what these kernels keep.
static bool mul_row_wins(const cg_ctx *c, size_t rows, bool cached)
{
    if (c->logn > 13 || c->k > 3) return false;
    if (c->dry) return c->dry_rows;
    return rounds_pay(c, rows, c->logn == 13 ? IdleLimits{128, cached ? 192 : 128, 256}
                             : c->k == 3 ? IdleLimits{102, 176, 256} : IdleLimits{128, 256, 256});
}
// ks_row_kernel.  A rotation gains less than a relinearisation: its digits are scattered through LDS, with two barriers
// each and nothing else on the unit to fill them, where the mod-up launch has two workgroups to a unit.  us with the mod-down and
// another key on every call, three launches / two, rotation and relinearisation.  N = 8192, three digits: 32 units (128 compute
// units idle) 37.4 / 45.2 and 36.3 / 38.9, 33 (124): relinearisation 44.5 / 39.0, 42 (88): 47.8 / 46.2 and 46.6 / 41.0, 44 (80): 52.1 / 46.5, 48: 52.6 / 47.4
// and 51.3 / 42.2, 80 (192): 81.3 / 83.8, 96 (128): 91.9 / 87.2 and 89.5 / 81.3, 97 (124): 100.6 / 90.8, 129 (252): 129 / 129 and 128 / 118, 141 (204): 134 / 131, 193:
// 186 / 173.  Two digits at N = 8192: 42 units (130 idle) 31.4 / 37.4 and 30.4 / 32.8, 43 (127): 40.1 / 33.2, 44 (124): 42.6 / 36.9, 100 (212): 63.3 / 68.1, 128 (128): 74.0 / 71.3 and
// 73.6 / 67.6.  N = 4096, two digits: 43 (127) 24.5 / 25.2 and 23.0 / 21.9, 44 (124): 27.9 / 25.2, 88 (248): 33.1 / 34.8 and 31.9 / 32.2, 107 (191): 34.3 / 35.7
// and 33.5 / 32.3, 128 (128): 37.3 / 37.2, 131: 46 / 38; three digits: 34 (120) 30.4 / 31.0, 42 (88): 29.9 / 31.1, 44 (80): 30.9 / 31.0.
// Older than these figures, N = 8192: the second round's limit for relinearisations, which gain throughout (three digits, 65 units, 252 idle, 75.9 / 72.5, 80: 81.6 / 77.1, 90: 88.3 / 79.7;
// two, 86 (254): 59.3 / 59.1, 107 (191): 67.2 / 62.0), and the rotations' with three digits, even from 36 units (112 idle, 46.2 / 45.2) and from 90 (152, 90.5 / 87.8) on.
static bool ks_row_wins(const cg_ctx *c, size_t rows, bool rotation)
{
    if (c->logn > 13 || c->alpha != 1) return false;
    if (c->dry) return c->dry_rows;
    const int one = !rotation ? 127 : c->dnum <= 2 ? 124 : 84;
    return rounds_pay(c, rows, c->logn == 13 ? IdleLimits{one, rotation ? 127 : 128, rotation ? 204 : 256}
                                             : IdleLimits{one, rotation ? 140 : 256, 256});
}

// Transforms of the operands, tensor product and inverse transforms in one launch: x in coefficients, y in
// coefficients or (A.yhat) transformed; x_cts, y_cts distinct ciphertexts of each
template <bool HAT>
static int launch_mul_row(cg_ctx *c, hipStream_t s, const MulRowArgs &A, double *tens, uint32_t batch, double x_cts,
                          double y_cts)
{
    const bool half = c->logn == 14;
    const size_t nwg = (size_t)batch * c->KL * (half ? 2 : 1);
    const int x_rows = half ? c->KL : c->k, y_rows = HAT ? c->KL : x_rows;
    const double bytes = (double)limb_bytes(c) * (2.0 * x_rows * x_cts + 2.0 * y_rows * y_cts + 3.0 * c->KL * batch);
    ProfScope ps(c, s, KID_MULROW, bytes, (double)nwg);
#define CG_MULROW(LG, K)                                                                                   \
    do {                                                                                                  \
        const unsigned threads = (1u << LG) / 8;                                                          \
        const unsigned grid = ntt_grid<mul_row_kernel<LG, 8, K, HAT>>(c, nwg, (int)threads);              \
        if (c->dry) return CG_OK;                                                                         \
        return launch_kernel(mul_row_kernel<LG, 8, K, HAT>, dim3(grid), dim3(threads), s, A,              \
                             StTens<K == 0>{{tens, LG}}, (const double *)(K ? c->tw : c->tw2),            \
                             (const double *)(K ? c->itw : c->itw2), (const DevConst *)c->dc, (int)nwg);  \
    } while (0)
    if (c->logn == 14) CG_MULROW(13, 0);
    switch (c->logn * 10 + c->k) {
    case 121: CG_MULROW(12, 1);
    case 122: CG_MULROW(12, 2);
    case 123: CG_MULROW(12, 3);
    case 131: CG_MULROW(13, 1);
    case 132: CG_MULROW(13, 2);
    case 133: CG_MULROW(13, 3);
    default: return CG_EINVAL;
    }
#undef CG_MULROW
}
// Sums of products over groups of units in one launch; every group is taken in `parts` parts.  HAT: y transformed (N = 4096 and 16384)
template <bool HAT>
static int launch_mul_sum_row(cg_ctx *c, hipStream_t s, const MulRowArgs &A, double *tens, uint32_t groups, const SumParts &S)
{
    const bool half = c->logn == 14;
    const size_t nwg = (size_t)(S.ranges ? S.ranges : groups * S.stride) * c->KL * (half ? 2 : 1);
    const double units = S.units;
    ProfScope ps(c, s, KID_MULSUMROW, (double)limb_bytes(c) * (4.0 * (half ? c->KL : c->k) * units + 3.0 * groups * S.stride * c->KL),
                 units * c->KL * (half ? 2 : 1));
#define CG_MULSUMROW(LG, K, H)                                                                             \
    do {                                                                                                  \
        const unsigned threads = (1u << LG) / 8;                                                          \
        const unsigned grid = ntt_grid<mul_sum_row_kernel<LG, 8, K, H>>(c, nwg, (int)threads);            \
        if (c->dry) return CG_OK;                                                                         \
        return launch_kernel(mul_sum_row_kernel<LG, 8, K, H>, dim3(grid), dim3(threads), s, A, S, \
                             StTens<K == 0>{{tens, LG}}, (const double *)(K ? c->tw : c->tw2), \
                             (const double *)(K ? c->itw : c->itw2), (const DevConst *)c->dc, (int)nwg);  \
    } while (0)
    if (half) CG_MULSUMROW(13, 0, HAT);
    switch (c->logn * 10 + c->k) {
    case 121: CG_MULSUMROW(12, 1, HAT);
    case 122: CG_MULSUMROW(12, 2, HAT);
    case 123: CG_MULSUMROW(12, 3, HAT);
    default: break;
    }
    if constexpr (!HAT) {
        switch (c->logn * 10 + c->k) {
        case 131: CG_MULSUMROW(13, 1, false);
        case 132: CG_MULSUMROW(13, 2, false);
        case 133: CG_MULSUMROW(13, 3, false);
        default: break;
        }
    }
    return CG_EINVAL;
#undef CG_MULSUMROW
}
// Whether that beats the launches of single transforms and a tensor inverse that walks over the group, and in how many
// parts.  In transforms of a row: six per unit and two besides in one launch, against four per row and unit spread
// over the chip, a half per unit of the group in every round of the tensor inverse, 1.2 besides, and a quarter on
// top for the traffic.  us at N = 8192, three primes, groups x units, three launches / one: 12 x 4 88 / 96, 12 x 2 60.5 / 62.3, 2 x 8 66.8 / 60.6, 8 x 8 112 / 98,
// 16 x 8 232 / 171, 3 x 8 81 / 62, 4 x 16 140 / 100, 8 x 100 1487 / 861; N = 4096, two primes: 12 x 4 43 / 39, 4 x 4 30.2 / 33.6, 16 x 4 44.6 / 52.6, 8 x 8 50.3 / 52.0,
// 12 x 8 61 / 50, 12 x 64 431 / 286.  The model is older than the kernel (a row's words asked for ahead, N^-1 in the scaling) and than sum_ranges, which it does not know of; it still takes three
// launches for 12 x 8 156 / 139, 6 x 8 97 / 95 and 12 x 16 324 / 248 (cut into ranges), at N = 4096 for 16 x 8 71 / 65, 9 x 12 75 / 67, 1 x 8 34.1 / 32.5 and 3 x 6 36.1 / 34.6.
//
// With one operand transformed already (hat) a unit has half the work in one launch, and two launches and an operand's way through
// memory fewer.  At N = 4096 that wins up to 5 n / 3 rows of (unit, prime), beyond which the other branches' launches fill the chip too
// and pieces as large as these no longer fit in beside them (decode step with a copy of the cache, two primes, heads x
// ciphertexts: 12 x 4 177 / 171, 8 x 8 197 / 182, 16 x 5 213 / 209, 12 x 7 214 / 211, 11 x 8 235 / 245, 15 x 6 242 / 250,
// 16 x 6 248 / 261, 14 x 7 250 / 277).  At N = 8192 the sums spill beside the transform: 1 x 1 187 / 201, 4 x 2 212 / 222,
// 12 x 4 423 / 438, 16 x 8 925 / 903.
static bool mul_sum_parts(const cg_ctx *c, uint32_t groups, uint32_t group, uint32_t &parts, bool hat = false)
{
    if (c->logn > (hat ? 12 : 13) || c->k > 3) return false;
    if (c->dry) return c->dry_rows;
    const double n = c->n_cu, base = (double)groups * c->KL;
    if (hat && 3.0 * base * group > 5.0 * n) return false;
    double best = 1e30;
    uint32_t best_parts = 1;
    for (uint32_t q = 1; q <= group && q <= 64; q++) {
        const double t = std::ceil(base * q / n) * ((hat ? 3.0 : 6.0) * ((group + q - 1) / q) + 2.0);
        if (t < best) { best = t; best_parts = q; }
    }
    if (!hat && best >= 1.25 * (4.0 * base * group / n + 0.5 * group * std::ceil(3.0 * base / n) + 1.2)) return false;
    parts = best_parts;
    return true;
}

// Parts of a group at N = 16384: as above, in transforms of a half row, four per unit (three with y transformed) and three
// besides; the fewest parts that are as fast, since scale_kernel reads every part.
// us of a context call with y transformed, six primes, heads x ciphertexts (all launches; keys the same in every call): a tensor
// inverse that walks over the group / mul_sum_row_kernel with three sums in registers, 16 of these spilled / with one in memory /
// mul_row_kernel with a part for every unit: 1 x 4 274 / 237 / 235 / 229, 3 x 2 296 / 278 / 275 / 270, 16 x 1 629 / 611 / 608 / 590;
// 4 x 4 348 / 327 / 327 / 339, 8 x 3 483 / 418 / 416 / 450, 16 x 3 784 / 722 / 709 / 750, 16 x 4 862 / 774 / 764 / 837.  The first
// three are those whose parts hold one unit each: nothing to sum, so do_mul has mul_row_kernel take these.
static uint32_t mul_sum_parts_half(const cg_ctx *c, uint32_t groups, uint32_t group, bool hat)
{
    const double n = c->n_cu, base = (double)groups * 2 * c->KL, per = hat ? 3.0 : 4.0;
    double best = 1e30;
    uint32_t parts = 1;
    for (uint32_t q = 1; q <= group && q <= 64; q++) {
        const double t = std::ceil(base * q / n) * (per * ((group + q - 1) / q) + 3.0);
        if (t < 0.97 * best) { best = t; parts = q; }
    }
    return parts;
}

// Sums of products with a transformed cache at N = 8192: the products one by one in mul_row_kernel, added up by scale_kernel, instead of the
// transforms of the operands and a tensor inverse that walks over the group.  us of a context alone, three primes, heads x ciphertexts (products x primes,
// 256 compute units): 16 x 1 (112) 178 / 179, 2 x 8 (112) 146 / 131, 3 x 6 (126) 143 / 135, 12 x 2 (168) 176 / 174, 14 x 2 (196) 191 / 178, 4 x 8 (224) 161 / 140,
// 8 x 4 (224) 163 / 157 (steps on both sides: 6 x 2 (84) 221 / 224, 9 x 4 (252) 368 / 375).  In a step only up to 2/3 of the units, which leaves the scores' some: 2 x 8 233 / 223,
// 5 x 4 (140) 258 / 256, 3 x 8 (168) 280 / 265, 6 x 4 283 / 278, but 14 x 2 356 / 356, 5 x 6 (210) 312 / 318, 8 x 4 333 / 337; and not where the scores are the
// longer chain, which it holds up (d2 = 128): 5 x 4 256 / 277, 7 x 3 (147) 270 / 290, 6 x 4 288 / 305; 2 x 8 237 / 231.
static bool mul_row_sums_win(const cg_ctx *c, size_t rows, const Beside &beside)
{
    const size_t n = (size_t)c->n_cu;
    if (c->logn != 13 || c->k > 3 || c->dry || beside.longer) return false;
    return 16 * rows >= 7 * n && (beside.others ? 3 * rows <= 2 * n : 8 * rows <= 7 * n);
}

// Ranges of units that end where groups do not (SumParts), one round of workgroups of them, where parts of whole groups
// would leave many workgroups idle: in the model above, a range that meets a second group has its transforms back twice
// (+ 4).  At N = 8192 and three primes, contexts of 8 groups of 128 units 1695 -> 1572 us, 10: 2021 -> 1910, 11: 2253 ->
// 2122, 16: 3250 -> 3061, 5: 1017 -> 997; 6, 9 and 12 groups, which parts fill as well, measure alike and stay.  At N = 4096, where two
// workgroups share a compute unit and fill each other's gaps, ranges lose: 97 -> 106 us for one group, 376 -> 404 for 12.
static bool sum_ranges(const cg_ctx *c, uint32_t groups, uint32_t group, SumParts &S)
{
    const int n = c->n_cu / c->KL, units = (int)(groups * group);
    if (c->dry || c->logn != 13 || n < 1) return false;
    const uint32_t parts = (uint32_t)S.stride;
    const double even = std::ceil((double)groups * parts * c->KL / c->n_cu) * (6.0 * ((group + parts - 1) / parts) + 2.0);
    if (6.0 * ((units + n - 1) / n) + 4.0 >= 0.99 * even) return false;
    // (a group of G units meets (G - 1) n / units + 2 ranges at most)
    const uint32_t most = (uint32_t)((uint64_t)(group - 1) * n / units) + 2;
    if (most > group) return false;
    S.stride = (int)most;
    S.ranges = n;
    return true;
}

// Algorithmic bytes (distinct inputs read once + outputs written once) are attached to every
// launch for the roofline report; LB = bytes of one residue row.
// b ciphertext of unit u sits at index (u / b_group) * b_stride + u % b_group (b_group = 0: dense)
static int do_mul(cg_ctx *c, hipStream_t s, const uint64_t *a2, const uint64_t *b2, uint64_t *out3,
                  uint32_t batch, uint32_t a_group, void *ws, int accumulate, uint32_t b_group = 0,
                  uint32_t b_stride = 0, const double *b_ext = nullptr, uint32_t sum_group = 0, const Beside &beside = {})
{
    // b_ext: the b operands are already in transformed extended-basis form (cg_cache_extend);
    // only the a operands are transformed here
    // sum_group: the tensor products of every sum_group consecutive units are summed before the
    // inverse transform and the scaling; out3 then holds batch / sum_group results
    const bool cached = b_group != 0;      // attention over a cache
    if (!b_group) { b_group = batch; b_stride = batch; }
    const uint32_t n_a = (batch + a_group - 1) / a_group;
    const uint32_t n_out = sum_group ? batch / sum_group : batch;
    const size_t polys = 2 * ((size_t)n_a + (b_ext ? 0 : batch));
    Bump w = bump(c, ws);
    double *ntt = w.take<double>(polys * c->KL);
    double *tens = w.take<double>((size_t)3 * c->KL * batch);
    const double LB = (double)limb_bytes(c), B = batch;
    MulSrc src{a2, b2, (int)n_a, (int)b_group, (int)b_stride, c->logn, 0};
    const int all = 1 << 30;
    uint32_t parts = 1;
    SumParts S{1, (int)(sum_group ? sum_group : 1), (int)batch, 0};
    if (c->logn == 14) {
        // operands lifted by a launch of its own, then half rows through the product in one launch: with a shared a
        // operand that is transformed once, or with the b operands given transformed, as the second operand
        const bool shared = a_group > 1 && !b_ext;
        MulRowArgs A{reinterpret_cast<const uint64_t *>(ntt), nullptr, b_ext, all, 0, (int)a_group, (int)b_group, (int)b_stride, 1,
                     2 * c->KL, 13};
        const size_t ct = (size_t)2 * c->KL * c->N;
        if (!b_ext) A.y = reinterpret_cast<const uint64_t *>(ntt + n_a * ct), A.y_group = all, A.y_stride = 0;
        if (shared) A = MulRowArgs{reinterpret_cast<const uint64_t *>(ntt + n_a * ct), nullptr, ntt, all, 0, 1, all, 0, (int)a_group,
                                   2 * c->KL, 13};
        CG_TRY(launch_lift(c, s, src, polys, ntt));
        if (shared) CG_TRY(launch_fwd_half(c, s, src, 2 * (size_t)n_a, ntt));
        if (sum_group) {
            CG_REQUIRE(a_group == 1);
            parts = mul_sum_parts_half(c, n_out, sum_group, b_ext != nullptr);
            // (while dry: the occupancy of the kernel that sums)
            if (b_ext && parts == sum_group && !c->dry) CG_TRY(launch_mul_row<true>(c, s, A, tens, batch, n_a, B));
            else {
                S.stride = (int)parts;
                CG_TRY(b_ext ? launch_mul_sum_row<true>(c, s, A, tens, n_out, S) : launch_mul_sum_row<false>(c, s, A, tens, n_out, S));
            }
        } else {
            CG_TRY(b_ext || shared ? launch_mul_row<true>(c, s, A, tens, batch, shared ? B : n_a, shared ? n_a : B)
                                   : launch_mul_row<false>(c, s, A, tens, batch, B, B));
        }
    } else if (sum_group && a_group == 1 && b_ext && mul_sum_parts(c, n_out, sum_group, parts, true)) {
        S.stride = (int)parts;
        CG_TRY(launch_mul_sum_row<true>(c, s, MulRowArgs{a2, nullptr, b_ext, all, 0, 1, (int)b_group, (int)b_stride, 1, c->k, c->logn},
                                        tens, n_out, S));
    } else if (sum_group && a_group == 1 && b_ext && mul_row_sums_win(c, (size_t)batch * c->KL, beside)) {
        parts = sum_group;
        CG_TRY(launch_mul_row<true>(c, s, MulRowArgs{a2, nullptr, b_ext, all, 0, 1, (int)b_group, (int)b_stride, 1, c->k, c->logn},
                                    tens, batch, B, B));
    } else if (sum_group && a_group == 1 && !b_ext && mul_sum_parts(c, n_out, sum_group, parts)) {
        S.stride = (int)parts;
        (void)sum_ranges(c, n_out, sum_group, S);
        CG_TRY(launch_mul_sum_row<false>(c, s, MulRowArgs{a2, b2, nullptr, all, 0, 1, (int)b_group, (int)b_stride, 1, c->k, c->logn},
                                         tens, n_out, S));
        parts = (uint32_t)S.stride;
    } else if (!sum_group && !(b_ext && a_group > 1) && mul_row_wins(c, (size_t)batch * c->KL, cached)) {
        MulRowArgs A{a2, b2, nullptr, all, 0, 1, (int)b_group, (int)b_stride, 1, c->k, c->logn};
        if (b_ext) {
            A.yhat = b_ext;
            CG_TRY(launch_mul_row<true>(c, s, A, tens, batch, B, B));
        } else if (a_group == 1) {
            CG_TRY(launch_mul_row<false>(c, s, A, tens, batch, B, B));
        } else {
            // the shared operand transformed once, the other one in the kernel
            CG_TRY(transform_ext(c, s, src, 2 * (size_t)n_a, ntt));
            A = MulRowArgs{b2, nullptr, ntt, (int)b_group, (int)b_stride, 1, all, 0, (int)a_group, c->k, c->logn};
            CG_TRY(launch_mul_row<true>(c, s, A, tens, batch, B, n_a));
        }
    } else {
        CG_TRY(transform_ext(c, s, src, polys, ntt));
        // tensor product fused into the inverse transform's load
        const LdInvTensor ld{ntt, b_ext, (int)a_group, (int)n_a, (int)b_group, (int)b_stride, c->logn};
        const size_t rows = (size_t)n_out * 3 * c->KL;
        const double tbytes = LB * c->KL * (2.0 * ((double)n_a + B) + 3.0 * n_out);
        if (sum_group) CG_TRY(launch_inv(c, s, rows, LdInvTensorSum{ld, (int)sum_group}, StTens<false>{{tens, c->logn}},
                                         KID_INV_TENSORSUM, tbytes));
        else CG_TRY(launch_inv(c, s, rows, ld, StTens<false>{{tens, c->logn}}, KID_INV_TENSOR, tbytes));
    }
    S.stride = (int)parts;
    const double sbytes = LB * (3.0 * c->KL * parts + 3.0 * c->k * (accumulate ? 2 : 1)) * n_out;
    const unsigned sblocks = pw_blocks(c, (size_t)n_out * 3);
#define CG_SCALE(K)                                                                                                  \
    do {                                                                                                             \
        if (c->logn == 14) CG_LAUNCH_PW(KID_SCALE, sbytes, (double)n_out, (scale_kernel<K, true>), sblocks, tens, out3, \
                                        S, accumulate, c->dc);                                              \
        else CG_LAUNCH_PW(KID_SCALE, sbytes, (double)n_out, (scale_kernel<K, false>), sblocks, tens, out3, S, \
                          accumulate, c->dc);                                                                        \
    } while (0)
    switch (c->k) {
    case 1: CG_SCALE(1); break;
    case 2: CG_SCALE(2); break;
    case 3: CG_SCALE(3); break;
    case 4: CG_SCALE(4); break;
    case 5: CG_SCALE(5); break;
    default: CG_SCALE(6); break;
    }
#undef CG_SCALE
    return CG_OK;
}

// Mod-up of one ring element per unit (src + b*src_stride, Galois map first when galois != 0): the
// dnum digits extended to the k+nsp primes and transformed, rows dig[b][dnum][k+nsp][N], canonical
static int launch_modup(cg_ctx *c, hipStream_t s, const uint64_t *src, size_t src_stride, uint32_t galois,
                        uint32_t batch, uint64_t *dig, bool whole = false)
{
    const size_t nrows = (size_t)batch * c->dnum * c->L;
    const double mbytes = (double)limb_bytes(c) * (c->k + (double)c->dnum * c->L) * batch;
    const StU64 st{dig, c->logn};
#define CG_MODUP(G, A) return launch_fwd(c, s, nrows, LdModup<G, A>{src, src_stride, galois, c->logn}, st, KID_FWD_MODUP, mbytes, whole ? 0 : row_parts(c, nrows, false))
    switch (c->alpha * 2 + (galois ? 1 : 0)) {
    case 2: CG_MODUP(false, 1);
    case 3: CG_MODUP(true, 1);
    case 4: CG_MODUP(false, 2);
    default: CG_MODUP(true, 2);
    }
#undef CG_MODUP
}

// the same behind a mod-down: in parts of rows, and with a map whole rows (no occupancy to look up: a workgroup takes one row)
static int launch_modup_down(cg_ctx *c, hipStream_t s, const LdModupDown<false> &ld, uint64_t *dig, size_t nrows, int parts)
{
    ProfScope ps(c, s, KID_FWD_MODUP, (double)limb_bytes(c) * (2.0 * c->k + 1.0 + c->L * c->dnum) * ((double)nrows / (c->L * c->dnum)), (double)nrows);
#define CG_MODUPDOWN(LG, LS)                                                                                                  \
    return launch_kernel(ntt_fwd_part_kernel<LG, LS, LdModupDown<false>, StU64>, dim3((unsigned)nrows << LS), dim3(1u << (LG - LS - 3)), s, \
                         ld, StU64{dig, c->logn}, (const double *)c->tw, (const DevConst *)c->dc, (int)nrows)
    switch (c->logn * 10 + parts) {
    case 121: CG_MODUPDOWN(12, 1);
    case 122: CG_MODUPDOWN(12, 2);
    case 132: CG_MODUPDOWN(13, 2);
    default: return CG_EINVAL;
    }
#undef CG_MODUPDOWN
}
static int launch_modup_down(cg_ctx *c, hipStream_t s, const LdModupDown<true> &ld, uint64_t *dig, size_t nrows)
{
    ProfScope ps(c, s, KID_FWD_MODUP, (double)limb_bytes(c) * (2.0 * c->k + 1.0 + c->L * c->dnum) * ((double)nrows / (c->L * c->dnum)), (double)nrows);
#define CG_MODUPDOWN(LG)                                                                                                      \
    return launch_kernel(ntt_fwd_kernel<LG, 8, LdModupDown<true>, StU64>, dim3((unsigned)nrows), dim3((1u << LG) / 8), s, ld,  \
                         StU64{dig, c->logn}, (const double *)c->tw, (const DevConst *)c->dc, (int)nrows)
    if (c->logn == 12) CG_MODUPDOWN(12);
    CG_MODUPDOWN(13);
#undef CG_MODUPDOWN
}
// inner product and inverse transforms, and the rows of the mod-down before
static int launch_ks_inner_after(cg_ctx *c, hipStream_t s, const uint64_t *dig, const double *key, double *acc, uint32_t batch, const ModdownArgs &A,
                                 const ModdownHoist &H)
{
    const size_t irows = (size_t)batch * 2 * c->L, pairs = (size_t)batch * c->k * c->N;
    const double dig_rows = (double)c->dnum * c->L;
    ProfScope ps(c, s, KID_INV_KSINNER, (double)limb_bytes(c) * ((dig_rows + 4.0 * c->L + 4.0 * c->k) * batch + 2.0 * dig_rows), (double)irows);
    const DevConst *dc = c->dc;
#define CG_INNERAFTER(LG, D)                                                                                                  \
    return launch_kernel(ks_inner_after_kernel<LG, 8, D>, dim3((unsigned)(irows + pairs / ((1u << LG) / 8))), dim3((1u << LG) / 8), s, \
                         LdInvKsInner<D>{dig, key, c->logn}, StInvF64{acc, c->logn}, (const double *)c->itw, (int)irows, A, H, dc)
    switch (c->logn * 10 + c->dnum) {
    case 121: CG_INNERAFTER(12, 1);
    case 122: CG_INNERAFTER(12, 2);
    case 123: CG_INNERAFTER(12, 3);
    case 131: CG_INNERAFTER(13, 1);
    case 132: CG_INNERAFTER(13, 2);
    case 133: CG_INNERAFTER(13, 3);
    default: return CG_EINVAL;
    }
#undef CG_INNERAFTER
}
// mod-up, inner product with the key and inverse transforms in one launch
static int launch_ks_row(cg_ctx *c, hipStream_t s, const uint64_t *src, size_t src_stride, uint32_t galois,
                         const double *key, double *acc, uint32_t batch)
{
    const size_t nwg = (size_t)batch * c->L;
    const double bytes = (double)limb_bytes(c) * ((c->k + 2.0 * c->L) * batch + 2.0 * c->dnum * c->L);
    ProfScope ps(c, s, KID_KSROW, bytes, (double)nwg);
#define CG_KSROW(LG, G)                                                                                       \
    do {                                                                                                     \
        const unsigned threads = (1u << LG) / 8;                                                             \
        const unsigned grid = ntt_grid<ks_row_kernel<LG, 8, G>>(c, nwg, (int)threads);                       \
        if (c->dry) return CG_OK;                                                                            \
        return launch_kernel(ks_row_kernel<LG, 8, G>, dim3(grid), dim3(threads), s,                          \
                             LdModup<G, 1>{src, src_stride, galois, c->logn}, key, StInvF64{acc, c->logn},   \
                             (const double *)c->tw, (const double *)c->itw, (const DevConst *)c->dc, (int)nwg); \
    } while (0)
    switch (c->logn * 2 + (galois ? 1 : 0)) {
    case 24: CG_KSROW(12, false);
    case 25: CG_KSROW(12, true);
    case 26: CG_KSROW(13, false);
    case 27: CG_KSROW(13, true);
    default: return CG_EINVAL;
    }
#undef CG_KSROW
}
// inner product with the key fused into the inverse transform's load
static int launch_ks_inner(cg_ctx *c, hipStream_t s, const uint64_t *dig, const double *key, double *acc, uint32_t batch)
{
    const size_t irows = (size_t)batch * 2 * c->L;
    const double dig_rows = (double)c->dnum * c->L;
    const double ibytes = (double)limb_bytes(c) * ((dig_rows + 2.0 * c->L) * batch + 2.0 * dig_rows);
    const StInvF64 ist{acc, c->logn};
#define CG_KSI(D) return launch_inv(c, s, irows, LdInvKsInner<D>{dig, key, c->logn}, ist, KID_INV_KSINNER, ibytes)
    switch (c->dnum) {
    case 1: CG_KSI(1);
    case 2: CG_KSI(2);
    case 3: CG_KSI(3);
    case 4: CG_KSI(4);
    case 5: CG_KSI(5);
    default: CG_KSI(6);
    }
#undef CG_KSI
}
// key switch of one ring element per unit (src + b*src_stride), then the final additions
static int do_keyswitch(cg_ctx *c, hipStream_t s, const uint64_t *src, size_t src_stride, uint32_t galois,
                        const double *key, uint64_t *out2, size_t out_stride, const uint64_t *add, size_t add_stride,
                        uint32_t galois_inv, int accumulate, uint32_t batch, void *ws,
                        const uint64_t *acc_add = nullptr, size_t acc_stride = 0, Beside beside = {})
{
    if (!acc_add) { acc_add = add; acc_stride = add_stride; }
    Bump w = bump(c, ws);
    uint64_t *dig = w.take<uint64_t>((size_t)c->dnum * c->L * batch);
    double *acc = w.take<double>((size_t)2 * c->L * batch);
    const double LB = (double)limb_bytes(c), B = batch;
    ModdownArgs A{acc, out2, out_stride, add, add_stride, galois_inv, accumulate, (int)batch, acc_add, acc_stride};
    const double add_rows = !add ? 0.0 : (galois_inv ? c->k + (accumulate ? 2.0 * c->k : 0.0) : 2.0 * c->k);
    if (add && ks_unit_wins(c, batch, 1, galois == 0)) {
        HoistTab T{};
        T.key[0] = key;
        return galois ? launch_ks_unit<KS_ROTATE>(c, s, src, src_stride, galois, T, A, ModdownHoist{}, acc, add_rows)
                      : launch_ks_unit<KS_PLAIN>(c, s, src, src_stride, galois, T, A, ModdownHoist{}, acc, add_rows);
    }
    if (!galois && ks_wide_wins(c, batch, true, beside)) {
        HoistTab T{};
        T.g[0] = 1;
        T.key[0] = key;
        CG_TRY(launch_ks_wide(c, s, src, src_stride, T, 1, acc, batch));
    } else if (ks_row_wins(c, (size_t)batch * c->L, galois != 0)) {
        CG_TRY(launch_ks_row(c, s, src, src_stride, galois, key, acc, batch));
    } else {
        CG_TRY(launch_modup(c, s, src, src_stride, galois, batch, dig, beside.crowd));
        CG_TRY(launch_ks_inner(c, s, dig, key, acc, batch));
    }
    return launch_moddown<false>(c, s, LB * (2.0 * c->L + add_rows + 2.0 * c->k) * B, batch, A, ModdownHoist{});
}

static int do_relin(cg_ctx *c, hipStream_t s, const uint64_t *in3, const void *rlk, uint64_t *out2, uint32_t batch,
                    void *ws, Beside beside = {})
{
    const size_t ct3 = (size_t)3 * c->k * c->N;
    return do_keyswitch(c, s, in3 + (size_t)2 * c->k * c->N, ct3, 0, static_cast<const double *>(rlk), out2,
                        (size_t)2 * c->k * c->N, in3, ct3, 0, 0, batch, ws, nullptr, 0, beside);
}

static uint32_t inv_mod_pow2(uint32_t g, uint32_t two_n)
{
    uint32_t x = g;   // Newton iteration: correct to 3 bits, doubles each step
    for (int i = 0; i < 5; i++) x *= 2 - g * x;
    return x & (two_n - 1);
}

// in_stride / out_stride: uint64 between consecutive units (0 = densely packed ciphertexts)
// out2 = rotate(in2, g) (accumulate = 0), in2 + rotate(in2, g) (accumulate = 1, acc_add null) or
// acc_add + rotate(in2, g) (accumulate = 1, acc_add given; out2 may be acc_add itself)
static int do_rotate(cg_ctx *c, hipStream_t s, const uint64_t *in2, uint32_t g, const void *gk, uint64_t *out2,
                     uint32_t batch, int accumulate, void *ws, size_t in_stride = 0, size_t out_stride = 0,
                     const uint64_t *acc_add = nullptr, size_t acc_stride = 0)
{
    const size_t ct2 = (size_t)2 * c->k * c->N;
    if (!in_stride) in_stride = ct2;
    if (!out_stride) out_stride = ct2;
    return do_keyswitch(c, s, in2 + (size_t)c->k * c->N, in_stride, g, static_cast<const double *>(gk), out2,
                        out_stride, in2, in_stride, inv_mod_pow2(g, 2u * c->N), accumulate, batch, ws, acc_add,
                        acc_stride);
}

// inner products, inverse transforms and mod-down of the rotations of a hoisted series in one launch
static int launch_rot_row(cg_ctx *c, hipStream_t s, const uint64_t *dig, const HoistTab &T, const ModdownArgs &A,
                          const ModdownHoist &H, uint32_t n_rot)
{
    const size_t nwg = (size_t)2 * H.rot_batch * n_rot;
    const double B = H.rot_batch;
    ProfScope ps(c, s, KID_ROTROW, (double)limb_bytes(c) * ((c->dnum * c->L + c->k) * B + 2.0 * c->dnum * c->L * n_rot +
                                                            2.0 * c->k * B * n_rot), (double)nwg);
#define CG_ROTROW(LG, D)                                                                                   \
    do {                                                                                                  \
        const unsigned threads = (1u << LG) / 8;                                                          \
        const unsigned grid = ntt_grid<rot_row_kernel<LG, 8, D>>(c, nwg, (int)threads);                               \
        if (c->dry) return CG_OK;                                                                         \
        return launch_kernel(rot_row_kernel<LG, 8, D>, dim3(grid), dim3(threads), s, dig, T, A, H,        \
                             (const double *)c->itw, (const DevConst *)c->dc, (int)nwg);                  \
    } while (0)
    switch (c->logn * 10 + c->dnum) {
    case 121: CG_ROTROW(12, 1);
    case 122: CG_ROTROW(12, 2);
    case 123: CG_ROTROW(12, 3);
    case 131: CG_ROTROW(13, 1);
    case 132: CG_ROTROW(13, 2);
    case 133: CG_ROTROW(13, 3);
    default: return CG_EINVAL;
    }
#undef CG_ROTROW
}
// From half as many workgroups as compute units on.  us with the mod-up, two launches / one.  N = 8192, three digits: one
// ciphertext, 31 rotations 37 / 55, 64: 57 / 57, 80: 70 / 58, 127: 94 / 62; 4 x 16: 54 / 57, 8 x 8: 53 / 59, 12 x 5: 53 / 59, 12 x 6:
// 65 / 60, 36 x 3: 91 / 65.  N = 4096, three digits: 8 x 8 32 / 35, 12 x 6: 37 / 36; two digits: 2 x 32 26.9 / 25.0, 8 x 8: 25.7 / 25.5.
static bool rot_row_wins(const cg_ctx *c, size_t units)
{
    if (c->logn > 13 || c->dnum > 3 || c->nsp != 1) return false;
    if (c->dry) return c->dry_rows;
    return c->dnum > 2 ? 4 * units > (size_t)c->n_cu : 4 * units >= (size_t)c->n_cu;
}

// A series of rotations of each of `batch` ciphertexts (in2 + b*in_stride): out2 + (b*out_per_b + i)
// ciphertexts receives rotation i (Galois element gs[i], prepared key keys[i]) in the hoisted form:
// one lift, extension and transform of the digits of c1, then per rotation a permuted inner
// product, inverse transforms and the mod-down with sigma_g(c0).  More than MAXROT rotations go in
// several rounds over the same digits.  ws: dnum (k+nsp) rows per ciphertext + 2 (k+nsp) rows per
// rotation of a round.
static int do_rotate_hoisted(cg_ctx *c, hipStream_t s, const uint64_t *in2, size_t in_stride, uint32_t n_rot,
                             const uint32_t *gs, const void *const *keys, uint64_t *out2, uint32_t out_per_b,
                             uint32_t batch, void *ws)
{
    const size_t ct2 = (size_t)2 * c->k * c->N;
    const double LB = (double)limb_bytes(c), B = batch;
    const double dig_rows = (double)c->dnum * c->L;
    const uint32_t round_max = n_rot < (uint32_t)MAXROT ? n_rot : (uint32_t)MAXROT;
    Bump w = bump(c, ws);
    uint64_t *dig = w.take<uint64_t>((size_t)c->dnum * c->L * batch);
    double *acc = w.take<double>((size_t)2 * c->L * batch * round_max);
    int rc;
    CG_TRY(launch_modup(c, s, in2 + (size_t)c->k * c->N, in_stride, 0, batch, dig));
    for (uint32_t i0 = 0; i0 < n_rot; i0 += MAXROT) {
        const uint32_t nr = n_rot - i0 < (uint32_t)MAXROT ? n_rot - i0 : (uint32_t)MAXROT;
        HoistTab T{};
        ModdownHoist H{};
        for (uint32_t i = 0; i < nr; i++) {
            T.g[i] = gs[i0 + i];
            T.key[i] = static_cast<const double *>(keys[i0 + i]);
            H.ginv[i] = inv_mod_pow2(gs[i0 + i], 2u * c->N);
        }
        H.rot_batch = (int)batch;
        H.out_per_b = (int)out_per_b;
        // galois != 0 marks the rotation form; the element itself comes from the table
        ModdownArgs A{acc, out2 + (size_t)i0 * ct2, ct2, in2, in_stride, 1u, 0, (int)((size_t)batch * nr), in2, in_stride};
        const size_t units = (size_t)batch * nr, irows = units * 2 * c->L;
        if (rot_row_wins(c, units)) {
            CG_TRY(launch_rot_row(c, s, dig, T, A, H, nr));
            continue;
        }
        const double ibytes = LB * (dig_rows * B + 2.0 * c->L * units + 2.0 * dig_rows * nr);
        const StInvF64 ist{acc, c->logn};
#define CG_KSH(D) rc = launch_inv(c, s, irows, LdInvKsInnerHoisted<D>{dig, T, (int)batch, c->logn}, ist, KID_INV_KSINNER, ibytes)
        switch (c->dnum) {
        case 1: CG_KSH(1); break;
        case 2: CG_KSH(2); break;
        case 3: CG_KSH(3); break;
        case 4: CG_KSH(4); break;
        case 5: CG_KSH(5); break;
        default: CG_KSH(6); break;
        }
#undef CG_KSH
        CG_TRY(rc);
        CG_TRY(launch_moddown<true>(c, s, LB * ((2.0 * c->L + 2.0 * c->k) * units + c->k * B), units, A, H));
    }
    return CG_OK;
}

// out2[b] = in2[b] + sum_i rotation i of in2[b] (Galois elements gs, prepared keys), the rotations
// hoisted and their key-switch accumulators summed before the one division by P.  in_stride /
// out_stride as in do_rotate.  ws: (dnum + 2)(k+nsp) rows per ciphertext.
static int do_rotate_sum(cg_ctx *c, hipStream_t s, const uint64_t *in2, size_t in_stride, uint32_t n_rot,
                         const uint32_t *gs, const void *const *keys, uint64_t *out2, size_t out_stride,
                         uint32_t batch, void *ws, Beside beside = {})
{
    const size_t ct2 = (size_t)2 * c->k * c->N;
    if (!in_stride) in_stride = ct2;
    if (!out_stride) out_stride = ct2;
    const double LB = (double)limb_bytes(c), B = batch;
    const double dig_rows = (double)c->dnum * c->L;
    Bump w = bump(c, ws);
    uint64_t *dig = w.take<uint64_t>((size_t)c->dnum * c->L * batch);
    double *acc = w.take<double>((size_t)2 * c->L * batch);
    HoistTab T{};
    ModdownHoist H{};
    for (uint32_t i = 0; i < n_rot; i++) {
        T.g[i] = gs[i];
        T.key[i] = static_cast<const double *>(keys[i]);
        H.ginv[i] = inv_mod_pow2(gs[i], 2u * c->N);
    }
    H.n_sum = (int)n_rot;
    const uint64_t *c1 = in2 + (size_t)c->k * c->N;
    ModdownArgs A{acc, out2, out_stride, in2, in_stride, 1u, 1, (int)batch, in2, in_stride};
    if (ks_unit_wins(c, batch, n_rot)) return launch_ks_unit<KS_SUM>(c, s, c1, in_stride, 0, T, A, H, acc, 2.0 * c->k);
    if (ks_wide_wins(c, batch, false, beside)) {
        CG_TRY(launch_ks_wide(c, s, c1, in_stride, T, n_rot, acc, batch));
    } else if (ks_sum_row_wins(c, batch)) {
        const bool down = ks_sum_down_wins(c, batch, n_rot);
        CG_TRY(launch_ks_sum_row(c, s, c1, in_stride, T, n_rot, acc, batch, down ? c->k : 0));
        if (down) {
            CG_TRY(launch_ks_sum_down(c, s, c1, in_stride, T, A, H));
            if (!c->dry) return CG_OK;
        }
    } else {
        const bool whole = beside.crowd;
        CG_TRY(launch_modup(c, s, c1, in_stride, 0, batch, dig, whole));
        const double sbytes = LB * ((dig_rows + 2.0 * c->L) * B + 2.0 * dig_rows * n_rot);
        CG_TRY(launch_ks_sum(c, s, sbytes, dig, T, n_rot, acc, batch, beside.others));
        const size_t irows = (size_t)batch * 2 * c->L;
        // few rows are transformed in parts, and so not in place: two digits' rows have room for the results
        const int parts = !whole && c->dnum >= 2 ? acc_parts(c, irows, beside.others) : 0;
        double *to = parts ? reinterpret_cast<double *>(dig) : acc;
        CG_TRY(launch_inv(c, s, irows, LdInvF64{acc, c->L, c->logn}, StInvF64{to, c->logn}, KID_INV_F64,
                          LB * 2.0 * irows, parts));
        A.acc = to;
    }
    // reads: the accumulators and the ciphertext (the permuted reads of c0 come from LDS)
    return launch_moddown_sum(c, s, LB * (2.0 * c->L + 4.0 * c->k) * B, batch, A, H);
}

static int do_add(cg_ctx *c, hipStream_t s, const uint64_t *a, const uint64_t *b, uint64_t *out, size_t rows)
{
    CG_LAUNCH_PW(KID_ADD, (double)limb_bytes(c) * 3.0 * rows, (double)rows, add_kernel, pw_blocks(c, rows), a, b, out, (int)rows,
                 c->dc);
    return CG_OK;
}

// One launch for all of them: a copy per ciphertext through the runtime takes 4.7 us each, one after the other (A V of 12 heads
// 2306 -> 2282 us a call; N = 4096, 6 heads 216 -> 208).
static int do_copy(cg_ctx *c, hipStream_t s, const uint64_t *src, size_t src_stride, uint64_t *dst, size_t dst_stride, uint32_t cts)
{
    const unsigned per = (unsigned)(2 * c->k * (c->N / (2 * PW_THREADS)));
    CG_LAUNCH_PW(KID_COPY, (double)limb_bytes(c) * 4.0 * c->k * cts, (double)cts, copy_kernel, cts * per, src, src_stride, dst,
                 dst_stride, (int)per);
    return CG_OK;
}

static bool ptrs_ok(std::initializer_list<const void *> ps)
{
    for (const void *p : ps) if (!p || !aligned16(p)) return false;
    return true;
}
static bool batch_ok(uint32_t batch) { return batch >= 1 && batch <= (1u << 16); }
static bool galois_ok(const cg_ctx *c, uint32_t g) { return (g & 1) && g > 0 && g < 2u * c->N; }

// ---------------------------------------------------------------------------
// public entry points
// ---------------------------------------------------------------------------
static int public_transform(cg_ctx *c, void *stream, const uint64_t *in, uint64_t *out, const uint32_t *idx,
                            uint32_t n_limbs, bool inverse)
{
    CG_REQUIRE(c && idx && ptrs_ok({in, out}) && n_limbs >= 1 && n_limbs <= c->tab_cap);
    hipStream_t s = static_cast<hipStream_t>(stream);
    // The usual pattern -- row i modulo prime i % period, as in stacked ring elements -- needs no
    // table.  Any other assignment is staged through a context-owned device buffer; that copy
    // is ordered on the caller's stream before the kernel.  The pattern is 0, 1, ... period - 1 and
    // then equal to itself shifted by a period: one block comparison, whatever the number of rows.
    uint32_t period = 0;
    while (period < n_limbs && period < (uint32_t)c->L && idx[period] == period) period++;
    const bool periodic =
        period && memcmp(idx, idx + period, (size_t)(n_limbs - period) * sizeof(uint32_t)) == 0;
    const uint32_t *tab = nullptr;
    if (!periodic) {
        for (uint32_t i = 0; i < n_limbs; i++) CG_REQUIRE(idx[i] < (uint32_t)c->L);
        // the table is copied from the caller's (pageable) host array when the call is made, not when
        // a captured graph replays: refuse that form on a capturing stream
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        CG_HIP(hipStreamIsCapturing(s, &cap));
        CG_REQUIRE(cap == hipStreamCaptureStatusNone);
        CG_HIP(hipMemcpyAsync(c->tab, idx, n_limbs * sizeof(uint32_t), hipMemcpyHostToDevice, s));
        tab = c->tab;
    }
    if (!inverse)
        return launch_fwd(c, s, n_limbs, LdRowsU64{in, tab, (int)period, c->logn}, StU64{out, c->logn}, KID_FWD_ROWS,
                          2.0 * limb_bytes(c) * n_limbs, row_parts(c, n_limbs, false));
    return launch_inv(c, s, n_limbs, LdInvU64{in, tab, (int)period, c->logn}, StInvU64{out, c->logn}, KID_INV_U64,
                      2.0 * limb_bytes(c) * n_limbs, row_parts(c, n_limbs, true));
}
extern "C" int cg_ntt_forward(cg_ctx *c, void *stream, const uint64_t *in, uint64_t *out, const uint32_t *idx,
                              uint32_t n_limbs)
{
    return public_transform(c, stream, in, out, idx, n_limbs, false);
}
extern "C" int cg_ntt_inverse(cg_ctx *c, void *stream, const uint64_t *in, uint64_t *out, const uint32_t *idx,
                              uint32_t n_limbs)
{
    return public_transform(c, stream, in, out, idx, n_limbs, true);
}

extern "C" int cg_ksk_prepare(cg_ctx *c, void *stream, const uint64_t *raw, void *ksk)
{
    CG_REQUIRE(c && ptrs_ok({raw, ksk}));
    return launch_fwd(c, static_cast<hipStream_t>(stream), (size_t)c->dnum * 2 * c->L,
                      LdRowsU64{raw, nullptr, c->L, c->logn}, StF64Red{static_cast<double *>(ksk), c->logn},
                      KID_FWD_ROWS, 4.0 * limb_bytes(c) * c->dnum * c->L);
}

extern "C" int cg_plain_prepare(cg_ctx *c, void *stream, const uint64_t *pt, void *plain, uint32_t batch)
{
    CG_REQUIRE(c && ptrs_ok({pt, plain}) && batch_ok(batch));
    return launch_fwd(c, static_cast<hipStream_t>(stream), (size_t)batch * c->k, LdPlain{pt, c->logn},
                      StF64Red{static_cast<double *>(plain), c->logn}, KID_FWD_PLAIN,
                      (double)limb_bytes(c) * batch * (1.0 + c->k));
}

extern "C" int cg_mul(cg_ctx *c, void *stream, const uint64_t *a2, const uint64_t *b2, uint64_t *out3,
                      uint32_t batch, uint32_t a_group, void *ws)
{
    CG_REQUIRE(c && ptrs_ok({a2, b2, out3, ws}) && batch_ok(batch) && a_group >= 1);
    return do_mul(c, static_cast<hipStream_t>(stream), a2, b2, out3, batch, a_group, ws, 0);
}

extern "C" int cg_mul_sum(cg_ctx *c, void *stream, const uint64_t *a2, const uint64_t *b2, uint64_t *out3,
                          uint32_t n_groups, uint32_t group_len, void *ws)
{
    CG_REQUIRE(c && ptrs_ok({a2, b2, out3, ws}) && n_groups >= 1 && group_len >= 1);
    CG_REQUIRE((uint64_t)n_groups * group_len <= (1u << 16));
    return do_mul(c, static_cast<hipStream_t>(stream), a2, b2, out3, n_groups * group_len, 1, ws, 0, 0, 0, nullptr,
                  group_len);
}

extern "C" int cg_relin(cg_ctx *c, void *stream, const uint64_t *in3, const void *rlk, uint64_t *out2,
                        uint32_t batch, void *ws)
{
    CG_REQUIRE(c && ptrs_ok({in3, rlk, out2, ws}) && batch_ok(batch));
    return do_relin(c, static_cast<hipStream_t>(stream), in3, rlk, out2, batch, ws);
}

extern "C" int cg_mul_relin(cg_ctx *c, void *stream, const uint64_t *a2, const uint64_t *b2, const void *rlk,
                            uint64_t *out2, uint32_t batch, uint32_t a_group, void *ws)
{
    CG_REQUIRE(c && ptrs_ok({a2, b2, rlk, out2, ws}) && batch_ok(batch) && a_group >= 1);
    hipStream_t s = static_cast<hipStream_t>(stream);
    Bump w = bump(c, ws);
    uint64_t *d3 = w.take<uint64_t>((size_t)3 * c->k * batch);
    CG_TRY(do_mul(c, s, a2, b2, d3, batch, a_group, w.p, 0));
    return do_relin(c, s, d3, rlk, out2, batch, w.p);
}

extern "C" size_t cg_static_scratch_bytes(void) { return CG_STATIC_SCRATCH_BYTES; }

// cg_mul_relin on the library's own scratch array: no allocation, by this call or by anything it
// calls (launches and, with profiling on, event records only)
extern "C" int cg_mul_relin_static(cg_ctx *c, void *stream, const uint64_t *a2, const uint64_t *b2, const void *rlk,
                                   uint64_t *out2, uint32_t batch, uint32_t a_group)
{
    CG_REQUIRE(c && ptrs_ok({a2, b2, rlk, out2}) && batch_ok(batch) && a_group >= 1);
    if (cg_workspace_bytes(c, batch) > (size_t)CG_STATIC_SCRATCH_BYTES) return CG_ESCRATCH;
    int dev = -1;
    CG_HIP(hipGetDevice(&dev));
    CG_REQUIRE(dev == c->device && c->static_ws);   // the array's address differs from GPU to GPU
    return cg_mul_relin(c, stream, a2, b2, rlk, out2, batch, a_group, c->static_ws);
}

extern "C" int cg_rotate(cg_ctx *c, void *stream, const uint64_t *in2, uint32_t g, const void *gk, uint64_t *out2,
                         uint32_t batch, int accumulate, void *ws)
{
    CG_REQUIRE(c && ptrs_ok({in2, gk, out2, ws}) && batch_ok(batch) && galois_ok(c, g));
    CG_REQUIRE(!overlap(in2, out2, (size_t)batch * 2 * c->k * limb_bytes(c)));
    return do_rotate(c, static_cast<hipStream_t>(stream), in2, g, gk, out2, batch, accumulate, ws);
}

static bool rot_series_ok(const cg_ctx *c, uint32_t n_rot, const uint32_t *gs, const void *const *keys)
{
    if (!gs || !keys || n_rot < 1 || n_rot > 4096) return false;
    for (uint32_t i = 0; i < n_rot; i++)
        if (!galois_ok(c, gs[i]) || !keys[i] || !aligned16(keys[i])) return false;
    return true;
}

extern "C" int cg_rotate_hoisted(cg_ctx *c, void *stream, const uint64_t *in2, uint32_t n_rot, const uint32_t *gs,
                                 const void *const *gks, uint64_t *out2, uint32_t batch, void *ws)
{
    CG_REQUIRE(c && ptrs_ok({in2, out2, ws}) && batch_ok(batch) && rot_series_ok(c, n_rot, gs, gks));
    CG_REQUIRE((uint64_t)batch * n_rot <= (1u << 16));
    const size_t ct2b = (size_t)2 * c->k * limb_bytes(c);
    CG_REQUIRE(!overlap(in2, ct2b * batch, out2, ct2b * batch * n_rot));
    return do_rotate_hoisted(c, static_cast<hipStream_t>(stream), in2, (size_t)2 * c->k * c->N, n_rot, gs, gks, out2,
                             n_rot, batch, ws);
}

extern "C" int cg_rotate_sum_hoisted(cg_ctx *c, void *stream, const uint64_t *in2, uint32_t n_rot, const uint32_t *gs,
                                     const void *const *gks, uint64_t *out2, uint32_t batch, void *ws)
{
    CG_REQUIRE(c && ptrs_ok({in2, out2, ws}) && batch_ok(batch) && rot_series_ok(c, n_rot, gs, gks));
    CG_REQUIRE(n_rot <= (uint32_t)MAXROT);
    const size_t ct2b = (size_t)2 * c->k * limb_bytes(c);
    CG_REQUIRE(!overlap(in2, ct2b * batch, out2, ct2b * batch));
    return do_rotate_sum(c, static_cast<hipStream_t>(stream), in2, 0, n_rot, gs, gks, out2, 0, batch, ws);
}

extern "C" int cg_add(cg_ctx *c, void *stream, const uint64_t *a, const uint64_t *b, uint64_t *out, uint32_t ncomp,
                      uint32_t batch)
{
    CG_REQUIRE(c && ptrs_ok({a, b, out}) && batch_ok(batch) && (ncomp == 2 || ncomp == 3));
    return do_add(c, static_cast<hipStream_t>(stream), a, b, out, (size_t)batch * ncomp * c->k);
}

extern "C" int cg_add_plain(cg_ctx *c, void *stream, const uint64_t *in2, const uint64_t *pt, uint32_t n_plain,
                            int negative, uint64_t *out2, uint32_t batch)
{
    CG_REQUIRE(c && ptrs_ok({in2, pt, out2}) && batch_ok(batch) && n_plain >= 1 && n_plain <= batch);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const size_t rows = (size_t)batch * 2 * c->k;
    CG_LAUNCH_PW(KID_ADD, (double)limb_bytes(c) * (2.0 * rows + n_plain), (double)rows, add_plain_kernel, pw_blocks(c, rows), in2, pt,
                 out2, (int)batch, (int)n_plain, negative ? 1 : 0, c->dc);
    return CG_OK;
}

extern "C" int cg_mul_plain(cg_ctx *c, void *stream, const uint64_t *in2, const void *plain, uint32_t plain_stride,
                            uint64_t *out2, uint32_t batch, void *ws)
{
    CG_REQUIRE(c && ptrs_ok({in2, plain, out2, ws}) && batch_ok(batch));
    hipStream_t s = static_cast<hipStream_t>(stream);
    const size_t rows = (size_t)batch * 2 * c->k;
    return launch_mulplain(c, s, rows, in2, static_cast<const double *>(plain), (int)plain_stride, 0,
                           StInvU64{out2, c->logn},
                           (double)limb_bytes(c) * (2.0 * rows + c->k * (plain_stride ? (double)batch : 1.0)));
}

extern "C" int cg_kv_append(cg_ctx *c, void *stream, uint64_t *cache, uint32_t cache_stride_cts, uint32_t n_caches,
                            uint32_t tau, const uint64_t *rows_dev, const void *masks, uint32_t d2, void *ws)
{
    CG_REQUIRE(c && ptrs_ok({cache, rows_dev, masks, ws}) && batch_ok(n_caches));
    CG_REQUIRE(d2 >= 1 && (d2 & (d2 - 1)) == 0 && d2 <= (uint32_t)c->N / 2);
    const uint32_t B = (uint32_t)c->N / d2, ct_idx = tau / B, blk = tau % B;
    CG_REQUIRE(ct_idx < cache_stride_cts);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const size_t rows = (size_t)n_caches * 2 * c->k;
    const size_t ct2 = (size_t)2 * c->k * c->N;
    return launch_mulplain(c, s, rows, rows_dev, static_cast<const double *>(masks), 0, (int)blk,
                           StInvAppend{cache + (size_t)ct_idx * ct2, (size_t)cache_stride_cts * ct2,
                                       blk == 0 ? 1 : 0, c->logn},
                           (double)limb_bytes(c) * ((blk == 0 ? 2.0 : 3.0) * rows + c->k));
}

static bool pow2_d(const cg_ctx *c, uint32_t d2) { return d2 >= 2 && (d2 & (d2 - 1)) == 0 && d2 <= (uint32_t)c->N / 4; }
static uint32_t pow3_mod(uint32_t e, uint32_t two_n)
{
    uint64_t r = 1, b = 3;
    for (; e; e >>= 1, b = b * b % two_n)
        if (e & 1) r = r * b % two_n;
    return (uint32_t)r;
}

// A relinearisation (in3; null: x0 holds what the first rotation takes) and a chain of single rotations, each added to what it rotates: a rotation's mod-up
// takes the mod-down before it in its loader, and that mod-down's rows come with the rotation's inner products (ks_inner_after_kernel), two launches a rotation instead
// of three.  Taken while the mod-up has no more rows than compute units, at N = 4096 (two workgroups to a unit) one and a half times as many.  Beside scores whose mod-ups
// have a row for every unit only a context that leads: the step waits for its chain, and the scores' work fits in beside it.  us a step, three launches / two, heads x
// ciphertexts, d2 = 64 unless said.  N = 8192, three primes: 1 x 1 267 / 239, 4 x 2 302 / 277, 9 x 1 317 / 298, 12 x 1 354 / 311, 16 x 1 394 / 371, 5 x 4 374 / 350, 8 x 2
// (d2 = 128) 352 / 318, 7 x 3 393 / 362; above, with a limit at 3/2: 11 x 2 406 / 421, 10 x 3 480 / 498, 8 x 3 415 / 410.  N = 4096, two: 1 x 1 239 / 200, 10 x 2 243 / 198,
// 16 x 1 240 / 192, 11 x 4 278 / 260, 12 x 5 297 / 286, 16 x 4 306 / 299, and at twice the units 16 x 5 317 / 336.  A context beside more scores: d2 = 32 (eight rotations
// against five) 12 x 4 621 / 561, 10 x 3 489 / 437, 5 x 7 510 / 470, 16 x 4 733 / 724, N = 4096 11 x 4 290 / 245, 16 x 5 323 / 297; with more than a round of (unit,
// prime) 14 x 8 1033 / 1054, N = 4096 16 x 8 403 / 408; seven rotations against six 16 x 2 517 / 532, 5 x 7 504 / 515, 8 x 5 594 / 572.  Projections of a token, a
// chain of eight rotations of 1, 4, 9, 16 and 21 units: N = 8192 198 / 163, 202 / 177, 236 / 195, 248 / 203, 249 / 228, N = 4096, seven, 112 / 89 to 136 / 114, 36 units 147 / 123.
// The launch of inner products and mod-down holds on to the end of a chain of fewer digits, whose mod-up has few rows: up to three of its workgroups to a unit at N = 8192, 5 1/2 at
// N = 4096, 3 3/4 with one rotation.  Scores or context alone, d2 = 64: one prime 48 units 236 / 212, 64 259 / 251, 100 335 / 356, 128 355 / 404; two 30 260 / 246, 34 271 / 261,
// context of 42 337 / 346; N = 4096, one 96 197 / 186, projection of 128 175 / 178; two, one rotation, 42 74.9 / 71.9, 64 98.5 / 105.  In a step, with other numbers of digits than
// three at N = 8192 and two at N = 4096, up to 9/4: one prime 48 x 1 355 / 353, 64 x 1 426 / 438; two 24 x 1 373 / 356, 28 x 1 398 / 411; N = 4096, one 48 x 1 216 / 200, 96 x 1
// 284 / 302, three 20 x 1 250 / 227, 24 x 1 282 / 287.  Scores beside a context with a mod-up row for every unit, N = 4096, 48 x 1 296 / 306, 64 x 1 349 / 372.
static bool chain_joined_wins(const cg_ctx *c, uint32_t batch, int n, const Beside &beside)
{
    if (c->logn > 13 || c->alpha != 1 || c->nsp != 1 || c->dnum > 3 || !n || (beside.crowd && !beside.leads)) return false;
    const size_t cu = (size_t)c->n_cu, rows = (size_t)batch * c->dnum * c->L, blocks = (size_t)batch * (2 * c->L + 8 * c->k);
    if (beside.others && c->dnum != (c->logn == 12 ? 2 : 3)) return rows <= cu && 4 * blocks <= 9 * cu;
    if (c->logn == 12) return 2 * rows <= (beside.rows > cu ? 2 : 3) * cu && 4 * blocks <= (n == 1 ? 15 : 22) * cu;
    return rows <= cu && blocks <= 3 * cu;
}
// beside: whole rows in the first mod-up beside a crowd, as elsewhere: 10 x 3 440 / 435 (parts / whole rows), 4 x 8 415 / 402, 5 x 7 466 / 463, 8 x 5 546 / 552, with d2 = 32
static int chain_joined(cg_ctx *c, hipStream_t s, const uint64_t *in3, const void *rlk, uint64_t *x0, uint64_t *x1, uint64_t *out,
                        const uint32_t *gs, const void *const *keys, int n, uint32_t batch, void *ws, const Beside &beside = {})
{
    const size_t ct2 = (size_t)2 * c->k * c->N, ct3 = (size_t)3 * c->k * c->N, c1 = (size_t)c->k * c->N;
    const size_t nrows = (size_t)batch * c->dnum * c->L, irows = (size_t)batch * 2 * c->L;
    Bump w = bump(c, ws);
    uint64_t *dig = w.take<uint64_t>(nrows);
    double *acc[2] = {w.take<double>(irows), w.take<double>(irows)};
    ModdownArgs A{acc[0], x0, ct2, in3, ct3, 1u, 1, (int)batch, in3, ct3};
    ModdownHoist H{};
    if (in3) {
        CG_TRY(launch_modup(c, s, in3 + 2 * c1, ct3, 0, batch, dig, beside.crowd));
        CG_TRY(launch_ks_inner(c, s, dig, static_cast<const double *>(rlk), acc[0], batch));
    } else {
        CG_TRY(launch_modup(c, s, x0 + c1, ct2, gs[0], batch, dig));
        CG_TRY(launch_ks_inner(c, s, dig, static_cast<const double *>(keys[0]), acc[0], batch));
        A = ModdownArgs{acc[0], n == 1 ? out : x1, ct2, x0, ct2, 1u, 1, (int)batch, x0, ct2};
        H.ginv[0] = inv_mod_pow2(gs[0], 2u * c->N);
        H.n_sum = 1;
    }
    for (int i = in3 ? 0 : 1; i < n; i++) {
        double *to = A.acc == acc[0] ? acc[1] : acc[0];
        CG_TRY(launch_modup_down(c, s, LdModupDown<true>{A.acc, A.add + c1, A.add_stride, gs[i], c->logn}, dig, nrows));
        CG_TRY(launch_ks_inner_after(c, s, dig, static_cast<const double *>(keys[i]), to, batch, A, H));
        uint64_t *cur = A.out;
        A = ModdownArgs{to, i == n - 1 ? out : cur == x0 ? x1 : x0, ct2, cur, ct2, 1u, 1, (int)batch, cur, ct2};
        H.ginv[0] = inv_mod_pow2(gs[i], 2u * c->N);
        H.n_sum = 1;
    }
    return launch_moddown_sum(c, s, (double)limb_bytes(c) * (2.0 * c->L + 4.0 * c->k) * batch, batch, A, H);
}

// x <- x + rotate(x, g) for each g of the list, ping-ponging between two buffers;
// the last result lands in `out`.  x0 holds the start value.
static int rotate_add_chain(cg_ctx *c, hipStream_t s, uint64_t *x0, uint64_t *x1, uint64_t *out,
                            const uint32_t *gs, const void *const *keys, int n, uint32_t batch, void *ws, Beside beside = {})
{
    if (n > 1 && chain_joined_wins(c, batch, n, beside)) return chain_joined(c, s, nullptr, nullptr, x0, x1, out, gs, keys, n, batch, ws);
    uint64_t *cur = x0, *nxt = x1;
    for (int i = 0; i < n; i++) {
        uint64_t *dst = (i == n - 1) ? out : nxt;
        CG_TRY(do_rotate(c, s, cur, gs[i], keys[i], dst, batch, 1, ws));
        nxt = cur;
        cur = dst;
    }
    return CG_OK;
}

// A folding sum over the subset products of the generators gens[0 .. n_bits) taken in rounds:
// ceil(n_bits / w) rounds of as even a number of bits as possible, the longer ones first; a round
// over bits [b0, b0 + c) adds to its input its rotations by the 2^c - 1 products of non-empty
// subsets of gens[b0 .. b0 + c) (entry m - 1: the generators whose bit is set in m), hoisted, with
// one mod-down.  keys: the prepared keys of all rounds in that order.
struct FoldRounds {
    int n_rounds = 0, n_keys = 0;
    int first[16], count[16];
    std::vector<uint32_t> g;
};
static bool fold_rounds(const cg_ctx *c, const uint32_t *gens, int n_bits, uint32_t w, FoldRounds &R)
{
    if (w < 1 || w > 7 || n_bits < 0 || n_bits > 16) return false;   // 2^7 - 1 rotations fit one launch
    if (!n_bits) return true;
    const int rounds = (n_bits + (int)w - 1) / (int)w, lo = n_bits / rounds, extra = n_bits % rounds;
    int b0 = 0;
    for (int r = 0; r < rounds; r++) {
        const int cb = lo + (r < extra ? 1 : 0);
        R.first[r] = R.n_keys;
        R.count[r] = (1 << cb) - 1;
        for (uint32_t m = 1; m < (1u << cb); m++) {
            uint64_t e = 1;
            for (int i = 0; i < cb; i++)
                if ((m >> i) & 1) e = e * gens[b0 + i] % (2u * c->N);
            R.g.push_back((uint32_t)e);
        }
        R.n_keys += R.count[r];
        b0 += cb;
    }
    R.n_rounds = rounds;
    return true;
}
static bool fold_keys_ok(const FoldRounds &R, const void *const *keys)
{
    if (R.n_keys && !keys) return false;
    for (int i = 0; i < R.n_keys; i++)
        if (!keys[i] || !aligned16(keys[i])) return false;
    return true;
}
// x0 holds the start value; rounds ping-pong between x0 and x1, the last result lands in `out`
static int fold_chain(cg_ctx *c, hipStream_t s, uint64_t *x0, uint64_t *x1, uint64_t *out, const FoldRounds &R,
                      const void *const *keys, uint32_t batch, void *ws, Beside beside = {})
{
    uint64_t *cur = x0, *nxt = x1;
    for (int r = 0; r < R.n_rounds; r++) {
        uint64_t *dst = (r == R.n_rounds - 1) ? out : nxt;
        CG_TRY(do_rotate_sum(c, s, cur, 0, (uint32_t)R.count[r], R.g.data() + R.first[r], keys + R.first[r], dst, 0,
                             batch, ws, beside));
        nxt = cur;
        cur = dst;
    }
    return CG_OK;
}

// A relinearisation and the rounds behind it where few units leave every launch bound by its own latency: the mod-up of a round takes the mod-down
// before it in its loader, and that mod-down's rows come with the round's sums (ks_sum_after_kernel), three launches a round instead of four.  Every part of
// every row repeats the mod-down of its digit, so up to half a row of the mod-up per compute unit at N = 4096, a quarter at N = 8192 (quarters of rows, as
// row_parts).  us, four launches / three, steps as heads x ciphertexts (plain cache, with a transformed one).
// - The sums take one ciphertext a thread, with the mod-down's blocks behind them: up to three workgroups to a unit at N = 8192 (five in a step, whose other branch
//   waits as well), seven at N = 4096.  Alone, 3 bits a round: three primes, scores (d2 = 64) 2 units 94.9 / 91.0, 4 102 / 102, context (d2 = 2) 4 156 / 160, 5 166 / 171; one
//   prime, context (d2 = 64) 8 110 / 108, 16 122 / 128, 32 153 / 166; N = 4096, one 37 91.3 / 89.0, 64 95.1 / 103.  Steps: three primes 1 x 2 178 / 161, 179 / 168, 1 x 4 177 / 164,
//   181 / 172, 4 x 1 (d2 = 32) 176 / 166, 183 / 177, 5 x 1 176 / 173, 185 / 183; beyond 9 x 1 208 / 213, 216 / 221, 10 x 1 (d2 = 32) 215 / 229, 228 / 241; one 16 x 1 167 / 159, 24 x 1
//   173 / 184, 32 x 1 192 / 223; two 8 x 1 171 / 163, 10 x 1 172 / 173, 180 / 195.
// - Its keys stay in L2 (sum_keys_stay), also those of the other branch's rounds, whose sums it would hold up: context alone, d2 = 64, a round of 15 rotations, 2 units 102 / 99.9,
//   4 110 / 113, 5 117 / 123; steps of 4 bits 3 x 2 (d2 = 32) 169 / 168, 4 x 1 158 / 165, 4 x 2 174 / 183, 5 x 1 166 / 183, (d2 = 64) 159 / 177.
// - A step's context at N = 8192 only beside scores whose mod-ups have rows for 3/8 of the units: 4 x 2 181 / 176, 190 / 187, 4 x 4 221 / 220, 224 / 228, 5 x 4 254 / 259, 257 / 260; beside
//   longer scores for a quarter: d2 = 128, 5 x 1 179 / 168, 4 x 2 182 / 189, 2 x 4 (2 bits) 193 / 199.
// - N = 4096: both branches' mod-ups have rows for 7/8 of the units.  1 x 2 161 / 147, 10 x 1 174 / 156, 16 x 1 167 / 154, 163 / 153, 12 x 2 169 / 164, 151 / 154, 18 x 1 161 / 149, 148 / 155; beyond 20 x 1 140 / 148,
//   151 / 165, 10 x 3 147 / 151, 155 / 161, 16 x 2 154 / 161, 157 / 163 (on a host that launches more slowly 161 / 150, 165 / 158, 162 / 162).
static bool fold_joined_wins(const cg_ctx *c, uint32_t batch, const FoldRounds &R, const Beside &beside)
{
    if (c->logn > 13 || c->alpha != 1 || c->nsp != 1 || c->dnum > 3 || !R.n_rounds || beside.crowd) return false;
    const size_t cu = (size_t)c->n_cu, rows = (size_t)batch * c->dnum * c->L, per = (size_t)batch * (c->N / PW_THREADS), sums = per * c->L, down = per * c->k;
    if (sums + down > (c->logn == 12 ? 7 : beside.others ? 5 : 3) * cu) return false;
    if (c->logn == 12 ? beside.others && 8 * (beside.rows + rows) > 7 * cu : 8 * beside.rows > 3 * cu) return false;
    if (c->logn == 13 && beside.longer && 4 * beside.rows > cu) return false;
    if (!sum_keys_stay(c, sums, std::max(beside.most, (uint32_t)*std::max_element(R.count, R.count + R.n_rounds)), beside.others)) return false;
    return row_parts(c, rows, false) >= (c->logn == 13 ? 2 : 1);
}
static int fold_joined(cg_ctx *c, hipStream_t s, const uint64_t *in3, const void *rlk, uint64_t *x0, uint64_t *x1, uint64_t *out,
                       const FoldRounds &R, const void *const *keys, uint32_t batch, void *ws, Beside beside)
{
    const size_t ct2 = (size_t)2 * c->k * c->N, ct3 = (size_t)3 * c->k * c->N, c1 = (size_t)c->k * c->N;
    const size_t nrows = (size_t)batch * c->dnum * c->L, irows = (size_t)batch * 2 * c->L;
    const double LB = (double)limb_bytes(c), B = batch, dig_rows = (double)c->dnum * c->L;
    Bump w = bump(c, ws);
    uint64_t *dig = w.take<uint64_t>(nrows);
    double *acc = w.take<double>(irows), *sums = w.take<double>(irows);      // (ws_total has room for a product's rows here)
    const int parts = row_parts(c, nrows, false);
    ModdownArgs A{acc, x0, ct2, in3, ct3, 1u, 1, (int)batch, in3, ct3};
    ModdownHoist H{};
    CG_TRY(launch_modup(c, s, in3 + 2 * c1, ct3, 0, batch, dig));
    CG_TRY(launch_ks_inner(c, s, dig, static_cast<const double *>(rlk), acc, batch));
    for (int r = 0; r < R.n_rounds; r++) {
        const uint32_t n_rot = (uint32_t)R.count[r];
        HoistTab T{};
        for (uint32_t i = 0; i < n_rot; i++) {
            T.g[i] = R.g[R.first[r] + i];
            T.key[i] = static_cast<const double *>(keys[R.first[r] + i]);
        }
        CG_TRY(launch_modup_down(c, s, LdModupDown<false>{acc, A.add + c1, A.add_stride, 0, c->logn}, dig, nrows, parts));
        CG_TRY(launch_ks_sum_after(c, s, LB * ((dig_rows + 4.0 * c->L + 4.0 * c->k) * B + 2.0 * dig_rows * n_rot), dig, T, n_rot, sums, batch, A, H));
        CG_TRY(launch_inv(c, s, irows, LdInvF64{sums, c->L, c->logn}, StInvF64{acc, c->logn}, KID_INV_F64, LB * 2.0 * irows,
                          acc_parts(c, irows, beside.others)));
        uint64_t *cur = A.out;
        A = ModdownArgs{acc, r == R.n_rounds - 1 ? out : cur == x0 ? x1 : x0, ct2, cur, ct2, 1u, 1, (int)batch, cur, ct2};
        for (uint32_t i = 0; i < n_rot; i++) H.ginv[i] = inv_mod_pow2(T.g[i], 2u * c->N);
        H.n_sum = (int)n_rot;
    }
    return launch_moddown_sum(c, s, LB * (2.0 * c->L + 4.0 * c->k) * B, batch, A, H);
}

// generators of the two folding sums: the slots of a block (scores), the blocks and the two rows (context)
static int fold_generators(const cg_ctx *c, uint32_t d2, uint32_t *gs)
{
    int n = 0;
    for (uint32_t sh = 1; sh < d2; sh <<= 1) gs[n++] = pow3_mod(sh, 2u * c->N);
    return n;
}
static int block_generators(const cg_ctx *c, uint32_t d2, uint32_t *gs)
{
    int n = 0;
    for (uint32_t sh = d2; sh <= (uint32_t)c->N / 4; sh <<= 1) gs[n++] = pow3_mod(sh, 2u * c->N);
    gs[n++] = 2u * c->N - 1;
    return n;
}

extern "C" int cg_round_galois(const cg_ctx *c, int which, uint32_t d2, uint32_t round_bits, uint32_t *elts_host,
                               uint32_t cap, uint32_t *n_out)
{
    CG_REQUIRE(c && n_out && (which == 0 || which == 1) && pow2_d(c, d2) && (elts_host || !cap));
    uint32_t gs[20];
    const int nb = which ? block_generators(c, d2, gs) : fold_generators(c, d2, gs);
    FoldRounds R;
    CG_REQUIRE(fold_rounds(c, gs, nb, round_bits, R));
    for (uint32_t i = 0; i < cap && i < (uint32_t)R.n_keys; i++) elts_host[i] = R.g[i];
    *n_out = (uint32_t)R.n_keys;
    return CG_OK;
}

// kext != null: the cache in transformed form (kc is then not read)
// w != 0: the folding sum in rounds of w bits (fold_rounds), gk_fold holding the rounds' keys
static int scores_impl(cg_ctx *c, void *stream, const uint64_t *q, const uint64_t *kc, const double *kext,
                       uint32_t heads, uint32_t n_cts, uint32_t cache_stride_cts, uint32_t d2, const void *rlk,
                       const void *const *gk_fold, uint64_t *out, void *ws, uint32_t fold_w = 0, Beside beside = {})
{
    CG_REQUIRE(c && ptrs_ok({q, kext ? (const void *)kext : (const void *)kc, rlk, out, ws}) && gk_fold &&
               heads >= 1 && n_cts >= 1 && pow2_d(c, d2));
    CG_REQUIRE(cache_stride_cts >= n_cts);
    const uint32_t batch = heads * n_cts;
    CG_REQUIRE(batch_ok(batch));
    uint32_t gs[20];
    const int nrot = fold_generators(c, d2, gs);
    FoldRounds R;
    if (fold_w) {
        CG_REQUIRE(fold_rounds(c, gs, nrot, fold_w, R) && fold_keys_ok(R, gk_fold));
    } else {
        for (int i = 0; i < nrot; i++) CG_REQUIRE(gk_fold[i] && aligned16(gk_fold[i]));
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    Bump w = bump(c, ws);
    uint64_t *d3 = w.take<uint64_t>((size_t)3 * c->k * batch);
    uint64_t *xa = w.take<uint64_t>((size_t)2 * c->k * batch), *xb = w.take<uint64_t>((size_t)2 * c->k * batch);
    CG_TRY(do_mul(c, s, q, kc, d3, batch, n_cts, w.p, 0, n_cts, cache_stride_cts, kext));
    if (fold_w && fold_joined_wins(c, batch, R, beside)) return fold_joined(c, s, d3, rlk, xa, xb, out, R, gk_fold, batch, w.p, beside);
    if (!fold_w && chain_joined_wins(c, batch, nrot, beside)) return chain_joined(c, s, d3, rlk, xa, xb, out, gs, gk_fold, nrot, batch, w.p);
    CG_TRY(do_relin(c, s, d3, rlk, xa, batch, w.p, beside));
    if (fold_w) return fold_chain(c, s, xa, xb, out, R, gk_fold, batch, w.p, beside);
    return rotate_add_chain(c, s, xa, xb, out, gs, gk_fold, nrot, batch, w.p, beside);
}
extern "C" int cg_decode_scores(cg_ctx *c, void *stream, const uint64_t *q, const uint64_t *kc, uint32_t heads,
                                uint32_t n_cts, uint32_t cache_stride_cts, uint32_t d2, const void *rlk,
                                const void *const *gk_fold, uint64_t *out, void *ws)
{
    return scores_impl(c, stream, q, kc, nullptr, heads, n_cts, cache_stride_cts, d2, rlk, gk_fold, out, ws);
}
extern "C" int cg_decode_scores_ext(cg_ctx *c, void *stream, const uint64_t *q, const void *kext, uint32_t heads,
                                    uint32_t n_cts, uint32_t cache_stride_cts, uint32_t d2, const void *rlk,
                                    const void *const *gk_fold, uint64_t *out, void *ws)
{
    CG_REQUIRE(kext);
    return scores_impl(c, stream, q, nullptr, static_cast<const double *>(kext), heads, n_cts, cache_stride_cts, d2,
                       rlk, gk_fold, out, ws);
}

static int context_impl(cg_ctx *c, void *stream, const uint64_t *a, const uint64_t *vc, const double *vext,
                        uint32_t heads, uint32_t n_cts, uint32_t cache_stride_cts, uint32_t d2, const void *rlk,
                        const void *const *gk_block, uint64_t *out, void *ws, uint32_t fold_w = 0,
                        bool sum_first = false, Beside beside = {})
{
    CG_REQUIRE(c && ptrs_ok({a, vext ? (const void *)vext : (const void *)vc, rlk, out, ws}) && gk_block &&
               heads >= 1 && n_cts >= 1 && pow2_d(c, d2));
    CG_REQUIRE(cache_stride_cts >= n_cts);
    const uint32_t batch = heads * n_cts;
    CG_REQUIRE(batch_ok(batch));
    uint32_t gs[20];
    const int nrot = block_generators(c, d2, gs);
    FoldRounds R;
    if (fold_w) {
        CG_REQUIRE(fold_rounds(c, gs, nrot, fold_w, R) && fold_keys_ok(R, gk_block));
    } else {
        for (int i = 0; i < nrot; i++) CG_REQUIRE(gk_block[i] && aligned16(gk_block[i]));
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    Bump w = bump(c, ws);
    uint64_t *d3 = w.take<uint64_t>((size_t)3 * c->k * batch);
    uint64_t *y = w.take<uint64_t>((size_t)3 * c->k * heads);
    uint64_t *xa = w.take<uint64_t>((size_t)2 * c->k * heads), *xb = w.take<uint64_t>((size_t)2 * c->k * heads);
    if (sum_first) {
        // y[h] = one scaling of the sum over c of the tensor products
        CG_TRY(do_mul(c, s, a, vc, y, batch, 1, w.p, 0, n_cts, cache_stride_cts, vext, n_cts, beside));
    } else {
        CG_TRY(do_mul(c, s, a, vc, d3, batch, 1, w.p, 0, n_cts, cache_stride_cts, vext));
        // y[h] = sum_c d3[h][c]  (three components)
        const int rows = 3 * c->k;
        CG_LAUNCH_PW(KID_SUM_GROUPS, (double)limb_bytes(c) * rows * (batch + heads), (double)batch, sum_groups_kernel,
                     pw_blocks(c, (size_t)heads * rows), d3, y, (int)heads, (int)n_cts, rows, c->dc);
    }
    if (fold_w && fold_joined_wins(c, heads, R, beside)) return fold_joined(c, s, y, rlk, xa, xb, out, R, gk_block, heads, w.p, beside);
    if (!fold_w && chain_joined_wins(c, heads, nrot, beside)) return chain_joined(c, s, y, rlk, xa, xb, out, gs, gk_block, nrot, heads, w.p, beside);
    CG_TRY(do_relin(c, s, y, rlk, xa, heads, w.p, beside));
    if (fold_w) return fold_chain(c, s, xa, xb, out, R, gk_block, heads, w.p, beside);
    return rotate_add_chain(c, s, xa, xb, out, gs, gk_block, nrot, heads, w.p, beside);
}
extern "C" int cg_decode_context(cg_ctx *c, void *stream, const uint64_t *a, const uint64_t *vc, uint32_t heads,
                                 uint32_t n_cts, uint32_t cache_stride_cts, uint32_t d2, const void *rlk,
                                 const void *const *gk_block, uint64_t *out, void *ws)
{
    return context_impl(c, stream, a, vc, nullptr, heads, n_cts, cache_stride_cts, d2, rlk, gk_block, out, ws);
}
extern "C" int cg_decode_context_ext(cg_ctx *c, void *stream, const uint64_t *a, const void *vext, uint32_t heads,
                                     uint32_t n_cts, uint32_t cache_stride_cts, uint32_t d2, const void *rlk,
                                     const void *const *gk_block, uint64_t *out, void *ws)
{
    CG_REQUIRE(vext);
    return context_impl(c, stream, a, nullptr, static_cast<const double *>(vext), heads, n_cts, cache_stride_cts, d2,
                        rlk, gk_block, out, ws);
}

extern "C" int cg_decode_scores_hoisted(cg_ctx *c, void *stream, const uint64_t *q, const uint64_t *kc, const void *kext,
                                        uint32_t heads, uint32_t n_cts, uint32_t cache_stride_cts, uint32_t d2,
                                        uint32_t round_bits, const void *rlk, const void *const *gk_rounds,
                                        uint64_t *out, void *ws)
{
    CG_REQUIRE(round_bits >= 1);
    return scores_impl(c, stream, q, kext ? nullptr : kc, static_cast<const double *>(kext), heads, n_cts,
                       cache_stride_cts, d2, rlk, gk_rounds, out, ws, round_bits);
}
extern "C" int cg_decode_context_hoisted(cg_ctx *c, void *stream, const uint64_t *a, const uint64_t *vc, const void *vext,
                                         uint32_t heads, uint32_t n_cts, uint32_t cache_stride_cts, uint32_t d2,
                                         uint32_t round_bits, int sum_before_scaling, const void *rlk,
                                         const void *const *gk_rounds, uint64_t *out, void *ws)
{
    CG_REQUIRE(round_bits >= 1 && (sum_before_scaling == 0 || sum_before_scaling == 1));
    return context_impl(c, stream, a, vext ? nullptr : vc, static_cast<const double *>(vext), heads, n_cts,
                        cache_stride_cts, d2, rlk, gk_rounds, out, ws, round_bits, sum_before_scaling != 0);
}

extern "C" int cg_cache_extend(cg_ctx *c, void *stream, const uint64_t *cts, uint32_t n_groups, uint32_t group_len,
                               uint32_t group_stride_cts, void *ext)
{
    CG_REQUIRE(c && ptrs_ok({cts, ext}) && n_groups >= 1 && group_len >= 1 && group_stride_cts >= group_len);
    CG_REQUIRE((uint64_t)n_groups * group_len <= (1u << 16));
    const MulSrc src{nullptr, cts, 0, (int)group_len, (int)group_stride_cts, c->logn, 1};
    return transform_ext(c, static_cast<hipStream_t>(stream), src, (size_t)2 * n_groups * group_len,
                         static_cast<double *>(ext));
}

extern "C" size_t cg_decode_step_workspace_bytes(const cg_ctx *c, uint32_t heads, uint32_t n_cts)
{
    if (!c || !heads || !n_cts || (uint64_t)heads * n_cts > (1u << 16)) return 0;
    return 2 * cg_workspace_bytes(c, heads * n_cts) + cg_workspace_bytes(c, 2 * heads);
}

// ext != null: the cache's transformed copy is read by the products and brought up to date for
// the appended ciphertext of every cache
static int step_impl(cg_ctx *c, void *stream, const uint64_t *q, const uint64_t *a, uint64_t *cache, double *ext,
                     uint32_t heads, uint32_t n_cts, uint32_t cache_stride_cts, uint32_t d2, uint32_t tau,
                     const uint64_t *rows, const void *masks, const void *rlk, const void *const *gk_fold,
                     const void *const *gk_block, uint64_t *scores, uint64_t *context, void *ws,
                     uint32_t fold_w = 0, uint32_t block_w = 0, bool sum_first = false)
{
    CG_REQUIRE(c && ptrs_ok({q, a, cache, rows, masks, rlk, scores, context, ws}) && gk_fold && gk_block);
    CG_REQUIRE(heads >= 1 && n_cts >= 1 && batch_ok(heads * n_cts) && pow2_d(c, d2) && cache_stride_cts >= n_cts);
    CG_REQUIRE(tau / ((uint32_t)c->N / d2) < cache_stride_cts);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const size_t ct2 = (size_t)2 * c->k * c->N;
    uint64_t *vcache = cache + (size_t)heads * cache_stride_cts * ct2;
    char *ws_scores = static_cast<char *>(ws);
    char *ws_context = ws_scores + cg_workspace_bytes(c, heads * n_cts);
    char *ws_append = ws_context + cg_workspace_bytes(c, heads * n_cts);
    const size_t ext_ct = (size_t)2 * c->KL * c->N;          // doubles per transformed ciphertext
    const uint32_t app_idx = tau / ((uint32_t)c->N / d2);
    const double *kext = ext, *vext = ext ? ext + (size_t)heads * cache_stride_cts * ext_ct : nullptr;
    // append, then (with a transformed copy) re-transform the ciphertext every cache just received
    auto append = [&](hipStream_t st) -> int {
        CG_TRY(cg_kv_append(c, st, cache, cache_stride_cts, 2 * heads, tau, rows, masks, d2, ws_append));
        if (!ext) return CG_OK;
        return cg_cache_extend(c, st, cache + (size_t)app_idx * ct2, 2 * heads, 1, cache_stride_cts,
                               ext + (size_t)app_idx * ext_ct);
    };
    // The appended ciphertext is read by this step's products only when it lies inside the first
    // n_cts: then the append goes first on the caller's stream; otherwise it is a third branch.
    const bool append_first = tau / ((uint32_t)c->N / d2) < n_cts;
    if (append_first) CG_TRY(append(s));
    hipStream_t *side = s ? c->side_own : c->side_default;
    CG_HIP(hipEventRecord(c->ev_fork, s));
    CG_HIP(hipStreamWaitEvent(side[0], c->ev_fork, 0));
    if (!append_first) CG_HIP(hipStreamWaitEvent(side[1], c->ev_fork, 0));
    // Branches are always joined, also after a failed launch, so that the caller's stream never
    // runs ahead of work this call started.
    // One branch runs on the caller's stream, where it waits for no event and none waits for it, and is issued first: the scores, of n_cts times
    // the units, or the context, where it has more dependent key switches and the launches of both chains are short (few), or where the scores' key switches
    // (a workgroup per unit and prime) take one round and leave the context's mod-ups no room beside them (over: both together 5/4 of the compute
    // units and more), so that what is issued behind waits.  us a step with the scores there / the context, heads x ciphertexts (rows of the
    // scores + of the context's mod-ups): few, N = 8192, 8 x 1 (32) 212 / 202, 4 x 4 (64) 370 / 352, 16 x 2 (128) 378 / 370; N = 16384, 1 x 1
    // 278 / 262, 4 x 1 386 / 382, but 8 x 2 (128) 766 / 800.  over, N = 8192, three primes, rounds, with a transformed cache, chains:
    // 8 x 7 (224 + 96) 465 / 444, 447 / 432, 665 / 654; 10 x 5 (200 + 120) 442 / 436, 440 / 433, 643 / 648; 12 x 4 (192 + 144) 429 / 429,
    // 429 / 419, 640 / 632; 13 x 4 (208 + 156) 481 / 463, 476 / 463, 679 / 669; 16 x 4 (256 + 192) 531 / 523, 553 / 542, 763 / 752.  Below: 11 x 4 (176 + 132)
    // 407 / 431, 405 / 402, 632 / 633; 9 x 5 (180 + 108) 402 / 429, 389 / 390, 609 / 624; 6 x 8 (192 + 72) 395 / 400, 383 / 392, 573 / 587; beyond a round
    // of the scores 11 x 6 (264) 570 / 589, 563 / 574, 832 / 846; 12 x 6 (288) 594 / 619, 587 / 604, 873 / 883.  Two primes 14 x 6 (252 + 84) 471 / 442, 454 / 436,
    // 612 / 615; four 10 x 4 (200 + 200) 545 / 536, 527 / 522, 827 / 809, 7 x 5 (175 + 140) 457 / 492, 437 / 445, 683 / 701, but 11 x 3 (165 + 220) 559 / 575, 550 / 553,
    // 761 / 753; in digits of two primes 1 % either way.  N = 4096, where two workgroups share a unit, 8 x 8 (192 + 48) 198 / 185, 183 / 188, 305 / 301, 12 x 7 (252)
    // 225 / 233.  As many key switches in both (longer): N = 8192, rounds of 4 bits, 6 x 3 229 / 249, 4 x 4 with a transformed cache 208 / 223, 16 x 1 275 / 286,
    // but 2 x 4 181 / 169; N = 16384, d2 = 128, 2 x 3 407 / 430, 3 x 3 512 / 548, 4 x 3 666 / 679, but 1 x 1 282 / 270.  N = 4096 (d2 = 64), where the host's pace counts,
    // 10 x 3 156 / 149, 14 x 3 171 / 161, on a slower one 167 / 167, 172 / 167.  A key switch less than the scores (d2 = 128): chains 2 x 5 318 / 327.
    auto switches = [](uint32_t slots, uint32_t w) { const uint32_t bits = 31 - __builtin_clz(slots); return w ? (bits + w - 1) / w : bits; };
    const size_t srows = (size_t)heads * n_cts * c->L, own = (size_t)heads * c->dnum * c->L, n = (size_t)c->n_cu;
    const bool few = 8 * srows <= (c->logn == 14 ? 3 : 4) * n, over = c->logn == 13 && 4 * (srows + own) >= 5 * n && srows <= n;
    const uint32_t own_switches = switches(c->N / d2, block_w), their = switches(d2, fold_w);
    const bool longer = own_switches > their || (c->logn == 12 && own_switches == their), context_first = longer && (few || over);
    const size_t modups = (size_t)heads * n_cts * c->dnum * c->L;
    // rotations of the largest round
    auto most = [](uint32_t slots, uint32_t w, uint32_t rounds) { return w && rounds ? (1u << ((31 - __builtin_clz(slots) + rounds - 1) / rounds)) - 1 : 0u; };
    const Beside by_context{true, false, false, false, false, own, most(c->N / d2, block_w, own_switches)};
    const Beside by_scores{true, modups > n, fold_w && ks_wide_wins(c, heads * n_cts, false, by_context), their > own_switches, own_switches >= their + 2 && srows <= n,
                           modups, most(d2, fold_w, their)};
    auto scores_on = [&](hipStream_t st) {
        return scores_impl(c, st, q, cache, kext, heads, n_cts, cache_stride_cts, d2, rlk, gk_fold, scores, ws_scores, fold_w, by_context);
    };
    auto context_on = [&](hipStream_t st) {
        return context_impl(c, st, a, vcache, vext, heads, n_cts, cache_stride_cts, d2, rlk, gk_block, context, ws_context,
                            block_w, sum_first, by_scores);
    };
    int rc = context_first ? context_on(s) : scores_on(s);
    const int rc1 = context_first ? scores_on(side[0]) : context_on(side[0]);
    if (rc == CG_OK) rc = rc1;
    if (!append_first) {
        const int rc2 = append(side[1]);
        if (rc == CG_OK) rc = rc2;
    }
    for (int i = 0; i < (append_first ? 1 : 2); i++) {
        CG_HIP(hipEventRecord(c->ev_join[i], side[i]));
        CG_HIP(hipStreamWaitEvent(s, c->ev_join[i], 0));
    }
    return rc;
}

extern "C" int cg_decode_step(cg_ctx *c, void *stream, const uint64_t *q, const uint64_t *a, uint64_t *cache,
                              uint32_t heads, uint32_t n_cts, uint32_t cache_stride_cts, uint32_t d2, uint32_t tau,
                              const uint64_t *rows, const void *masks, const void *rlk, const void *const *gk_fold,
                              const void *const *gk_block, uint64_t *scores, uint64_t *context, void *ws)
{
    return step_impl(c, stream, q, a, cache, nullptr, heads, n_cts, cache_stride_cts, d2, tau, rows, masks, rlk, gk_fold,
                     gk_block, scores, context, ws);
}
extern "C" int cg_decode_step_ext(cg_ctx *c, void *stream, const uint64_t *q, const uint64_t *a, uint64_t *cache,
                                  void *cache_ext, uint32_t heads, uint32_t n_cts, uint32_t cache_stride_cts,
                                  uint32_t d2, uint32_t tau, const uint64_t *rows, const void *masks, const void *rlk,
                                  const void *const *gk_fold, const void *const *gk_block, uint64_t *scores,
                                  uint64_t *context, void *ws)
{
    CG_REQUIRE(cache_ext && aligned16(cache_ext));
    return step_impl(c, stream, q, a, cache, static_cast<double *>(cache_ext), heads, n_cts, cache_stride_cts, d2, tau,
                     rows, masks, rlk, gk_fold, gk_block, scores, context, ws);
}

extern "C" int cg_decode_step_hoisted(cg_ctx *c, void *stream, const uint64_t *q, const uint64_t *a, uint64_t *cache,
                                      void *cache_ext, uint32_t heads, uint32_t n_cts, uint32_t cache_stride_cts,
                                      uint32_t d2, uint32_t tau, const uint64_t *rows, const void *masks,
                                      const void *rlk, uint32_t fold_round_bits, const void *const *gk_fold_rounds,
                                      uint32_t block_round_bits, int sum_before_scaling,
                                      const void *const *gk_block_rounds, uint64_t *scores, uint64_t *context, void *ws)
{
    CG_REQUIRE(fold_round_bits >= 1 && block_round_bits >= 1 && (!cache_ext || aligned16(cache_ext)));
    CG_REQUIRE(sum_before_scaling == 0 || sum_before_scaling == 1);
    return step_impl(c, stream, q, a, cache, static_cast<double *>(cache_ext), heads, n_cts, cache_stride_cts, d2, tau,
                     rows, masks, rlk, gk_fold_rounds, gk_block_rounds, scores, context, ws, fold_round_bits,
                     block_round_bits, sum_before_scaling != 0);
}

extern "C" int cg_decode_scores_outer(cg_ctx *c, void *stream, const uint64_t *q, const uint64_t *kcols,
                                      uint32_t heads, uint32_t d2, const void *masks, const void *rlk,
                                      const void *const *gk_fold, uint64_t *out, void *ws)
{
    CG_REQUIRE(c && ptrs_ok({q, kcols, masks, rlk, out, ws}) && gk_fold && heads >= 1 && pow2_d(c, d2));
    const uint32_t batch = heads * d2;
    CG_REQUIRE(batch_ok(batch));
    int nrot = 0;
    uint32_t gs[16];
    for (uint32_t sh = 1; sh < d2; sh <<= 1) {
        CG_REQUIRE(gk_fold[nrot] && aligned16(gk_fold[nrot]));
        gs[nrot++] = pow3_mod(sh, 2u * c->N);
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    const double LB = (double)limb_bytes(c);
    Bump w = bump(c, ws);
    uint64_t *xa = w.take<uint64_t>((size_t)2 * c->k * batch), *xb = w.take<uint64_t>((size_t)2 * c->k * batch);
    uint64_t *d3 = w.take<uint64_t>((size_t)3 * c->k * batch);
    uint64_t *y = w.take<uint64_t>((size_t)3 * c->k * heads);
    // x[h][j] = q[h] * mask_j: one forward transform per query row, the mask product rides on the
    // inverse transform's load
    double *f = reinterpret_cast<double *>(d3);   // free until the products are formed
    const size_t qrows = (size_t)heads * 2 * c->k, xrows = (size_t)batch * 2 * c->k;
    CG_TRY(launch_fwd(c, s, qrows, LdRowsU64{q, nullptr, c->k, c->logn}, StF64{f, c->logn}, KID_FWD_ROWS,
                      LB * 2.0 * qrows));
    CG_TRY(launch_inv(c, s, xrows,
                      LdInvMulPlain{f, static_cast<const double *>(masks), (int)d2, (int)d2, 1, 0, c->logn},
                      StInvU64{xa, c->logn}, KID_INV_MULPLAIN, LB * (qrows + (double)d2 * c->k + xrows)));
    // broadcast q_j to every slot: log2(d2) rotate-and-add steps; the last one lands in xb or xa
    uint64_t *bc = (nrot & 1) ? xb : xa;
    if (nrot) CG_TRY(rotate_add_chain(c, s, xa, xb, bc, gs, gk_fold, nrot, batch, w.p));
    CG_TRY(do_mul(c, s, bc, kcols, d3, batch, 1, w.p, 0));
    const int rows = 3 * c->k;
    CG_LAUNCH_PW(KID_SUM_GROUPS, LB * rows * (batch + heads), (double)batch, sum_groups_kernel, pw_blocks(c, (size_t)heads * rows),
                 d3, y, (int)heads, (int)d2, rows, c->dc);
    return do_relin(c, s, y, rlk, out, heads, w.p);
}

extern "C" int cg_decode_context_outer(cg_ctx *c, void *stream, const uint64_t *a, const uint64_t *vcols,
                                       uint32_t heads, uint32_t d2, const void *rlk, const void *const *gk_all,
                                       uint64_t *out, void *ws)
{
    CG_REQUIRE(c && ptrs_ok({a, vcols, rlk, out, ws}) && gk_all && heads >= 1 && d2 >= 1);
    const uint32_t batch = heads * d2;
    CG_REQUIRE(batch_ok(batch));
    int nrot = 0;
    uint32_t gs[20];
    for (uint32_t sh = 1; sh <= (uint32_t)c->N / 4; sh <<= 1) gs[nrot++] = pow3_mod(sh, 2u * c->N);
    gs[nrot++] = 2u * c->N - 1;
    for (int i = 0; i < nrot; i++) CG_REQUIRE(gk_all[i] && aligned16(gk_all[i]));
    hipStream_t s = static_cast<hipStream_t>(stream);
    Bump w = bump(c, ws);
    uint64_t *d3 = w.take<uint64_t>((size_t)3 * c->k * batch);
    uint64_t *xa = w.take<uint64_t>((size_t)2 * c->k * batch), *xb = w.take<uint64_t>((size_t)2 * c->k * batch);
    CG_TRY(do_mul(c, s, a, vcols, d3, batch, d2, w.p, 0));
    CG_TRY(do_relin(c, s, d3, rlk, xa, batch, w.p));
    return rotate_add_chain(c, s, xa, xb, out, gs, gk_all, nrot, batch, w.p);
}

// kp[h][sigma*H + r] (m = 2H units per head): r = 0 copies of the source, K_r = rotate(K_{r-1}, 3^d2)
// sequentially for all heads at once, then the row-swapped copies (sigma = 1)
static int rotated_copies(cg_ctx *c, hipStream_t s, const uint64_t *src, uint32_t heads, uint32_t d2,
                          const void *gk_blk, const void *gk_swap, uint64_t *kp, void *ws)
{
    const uint32_t m = (uint32_t)c->N / d2, H = m / 2;
    const size_t ct2 = (size_t)2 * c->k * c->N;
    CG_TRY(do_copy(c, s, src, ct2, kp, m * ct2, heads));
    const uint32_t g_blk = pow3_mod(d2, 2u * c->N), g_swap = 2u * c->N - 1;
    for (uint32_t r = 1; r < H; r++)
        CG_TRY(do_rotate(c, s, kp + (size_t)(r - 1) * ct2, g_blk, gk_blk, kp + (size_t)r * ct2, heads, 0, ws,
                         (size_t)m * ct2, (size_t)m * ct2));
    for (uint32_t h = 0; h < heads; h++)
        CG_TRY(do_rotate(c, s, kp + (size_t)h * m * ct2, g_swap, gk_swap, kp + ((size_t)h * m + H) * ct2, H, 0, ws));
    return CG_OK;
}

// The same m copies per head, every one rotated out of the source itself as one series of hoisted
// rotations: unit sigma*H + r by 3^(d2 r), times 2N-1 for sigma = 1 (keys gk_copies[unit - 1])
static int rotated_copies_hoisted(cg_ctx *c, hipStream_t s, const uint64_t *src, uint32_t heads, uint32_t d2,
                                  const void *const *gk_copies, uint64_t *kp, void *ws)
{
    const uint32_t m = (uint32_t)c->N / d2, H = m / 2, two_n = 2u * c->N;
    const size_t ct2 = (size_t)2 * c->k * c->N;
    CG_TRY(do_copy(c, s, src, ct2, kp, m * ct2, heads));
    std::vector<uint32_t> gs(m - 1);
    for (uint32_t u = 1; u < m; u++) {
        const uint64_t g = pow3_mod(d2 * (u % H), two_n);
        gs[u - 1] = (uint32_t)(u >= H ? g * (two_n - 1) % two_n : g);
    }
    return do_rotate_hoisted(c, s, src, ct2, m - 1, gs.data(), gk_copies, kp + ct2, m, heads, ws);
}

// gk_copies != null: the copies of K come from hoisted rotations (gk_blk / gk_swap are then not used)
static int prefill_qk_impl(cg_ctx *c, void *stream, const uint64_t *q, const uint64_t *kk, uint32_t heads, uint32_t d2,
                           const void *rlk, const void *const *gk_fold, const void *gk_blk, const void *gk_swap,
                           const void *const *gk_copies, uint64_t *out, void *ws, uint32_t fold_w = 0)
{
    CG_REQUIRE(c && ptrs_ok({q, kk, rlk, out, ws}) && gk_fold && heads >= 1 && pow2_d(c, d2));
    const uint32_t m = (uint32_t)c->N / d2, batch = heads * m;
    CG_REQUIRE(batch_ok(batch));
    if (gk_copies) {
        for (uint32_t u = 1; u < m; u++) CG_REQUIRE(gk_copies[u - 1] && aligned16(gk_copies[u - 1]));
    } else {
        CG_REQUIRE(ptrs_ok({gk_blk, gk_swap}));
    }
    uint32_t gs[20];
    const int nrot = fold_generators(c, d2, gs);
    FoldRounds R;
    if (fold_w) {
        CG_REQUIRE(fold_rounds(c, gs, nrot, fold_w, R) && fold_keys_ok(R, gk_fold));
    } else {
        for (int i = 0; i < nrot; i++) CG_REQUIRE(gk_fold[i] && aligned16(gk_fold[i]));
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    // kp[h][sigma*H + r]: rotated copies of K, one ciphertext per output unit
    Bump w = bump(c, ws);
    uint64_t *kp = w.take<uint64_t>((size_t)2 * c->k * batch);
    uint64_t *xb = w.take<uint64_t>((size_t)2 * c->k * batch);
    uint64_t *d3 = w.take<uint64_t>((size_t)3 * c->k * batch);
    if (gk_copies) CG_TRY(rotated_copies_hoisted(c, s, kk, heads, d2, gk_copies, kp, w.p));
    else CG_TRY(rotated_copies(c, s, kk, heads, d2, gk_blk, gk_swap, kp, w.p));
    // all heads x m products at once
    CG_TRY(do_mul(c, s, q, kp, d3, batch, m, w.p, 0));
    CG_TRY(do_relin(c, s, d3, rlk, kp, batch, w.p));   // the rotated keys are consumed: reuse as x0
    if (fold_w) return fold_chain(c, s, kp, xb, out, R, gk_fold, batch, w.p);
    return rotate_add_chain(c, s, kp, xb, out, gs, gk_fold, nrot, batch, w.p);
}
extern "C" int cg_prefill_qk(cg_ctx *c, void *stream, const uint64_t *q, const uint64_t *kk, uint32_t heads,
                             uint32_t d2, const void *rlk, const void *const *gk_fold, const void *gk_blk,
                             const void *gk_swap, uint64_t *out, void *ws)
{
    return prefill_qk_impl(c, stream, q, kk, heads, d2, rlk, gk_fold, gk_blk, gk_swap, nullptr, out, ws);
}
extern "C" int cg_prefill_qk_hoisted(cg_ctx *c, void *stream, const uint64_t *q, const uint64_t *kk, uint32_t heads,
                                     uint32_t d2, uint32_t fold_round_bits, const void *rlk,
                                     const void *const *gk_fold, const void *const *gk_copies, uint64_t *out, void *ws)
{
    CG_REQUIRE(gk_copies);
    return prefill_qk_impl(c, stream, q, kk, heads, d2, rlk, gk_fold, nullptr, nullptr, gk_copies, out, ws,
                           fold_round_bits);
}

static int prefill_av_impl(cg_ctx *c, void *stream, const uint64_t *a, const uint64_t *v, uint32_t heads, uint32_t d2,
                           const void *rlk, const void *gk_blk, const void *gk_swap, const void *const *gk_copies,
                           uint64_t *out, void *ws, bool sum_first = false)
{
    CG_REQUIRE(c && ptrs_ok({a, v, rlk, out, ws}) && heads >= 1 && pow2_d(c, d2));
    const uint32_t m = (uint32_t)c->N / d2, batch = heads * m;
    CG_REQUIRE(batch_ok(batch));
    if (gk_copies) {
        for (uint32_t u = 1; u < m; u++) CG_REQUIRE(gk_copies[u - 1] && aligned16(gk_copies[u - 1]));
    } else {
        CG_REQUIRE(ptrs_ok({gk_blk, gk_swap}));
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    Bump w = bump(c, ws);
    uint64_t *vp = w.take<uint64_t>((size_t)2 * c->k * batch);
    uint64_t *d3 = w.take<uint64_t>((size_t)3 * c->k * batch);
    uint64_t *y = w.take<uint64_t>((size_t)3 * c->k * heads);
    if (gk_copies) CG_TRY(rotated_copies_hoisted(c, s, v, heads, d2, gk_copies, vp, w.p));
    else CG_TRY(rotated_copies(c, s, v, heads, d2, gk_blk, gk_swap, vp, w.p));
    if (sum_first) {
        CG_TRY(do_mul(c, s, a, vp, y, batch, 1, w.p, 0, 0, 0, nullptr, m));
    } else {
        CG_TRY(do_mul(c, s, a, vp, d3, batch, 1, w.p, 0));
        const int rows = 3 * c->k;
        CG_LAUNCH_PW(KID_SUM_GROUPS, (double)limb_bytes(c) * rows * (batch + heads), (double)batch, sum_groups_kernel,
                     pw_blocks(c, (size_t)heads * rows), d3, y, (int)heads, (int)m, rows, c->dc);
    }
    return do_relin(c, s, y, rlk, out, heads, w.p);
}
extern "C" int cg_prefill_av(cg_ctx *c, void *stream, const uint64_t *a, const uint64_t *v, uint32_t heads,
                             uint32_t d2, const void *rlk, const void *gk_blk, const void *gk_swap, uint64_t *out,
                             void *ws)
{
    return prefill_av_impl(c, stream, a, v, heads, d2, rlk, gk_blk, gk_swap, nullptr, out, ws);
}
extern "C" int cg_prefill_av_hoisted(cg_ctx *c, void *stream, const uint64_t *a, const uint64_t *v, uint32_t heads,
                                     uint32_t d2, int sum_before_scaling, const void *rlk,
                                     const void *const *gk_copies, uint64_t *out, void *ws)
{
    CG_REQUIRE(gk_copies && (sum_before_scaling == 0 || sum_before_scaling == 1));
    return prefill_av_impl(c, stream, a, v, heads, d2, rlk, nullptr, nullptr, gk_copies, out, ws,
                           sum_before_scaling != 0);
}

extern "C" int cg_prefill_repack(cg_ctx *c, void *stream, const uint64_t *x, uint32_t heads, uint32_t d2,
                                 const void *mask0, const void *const *gk_right, uint64_t *out, void *ws)
{
    CG_REQUIRE(c && ptrs_ok({x, mask0, out, ws}) && gk_right && heads >= 1 && pow2_d(c, d2));
    const uint32_t m = (uint32_t)c->N / d2, H = m / 2, batch = heads * m;
    CG_REQUIRE(batch_ok(batch));
    const uint32_t wdt = H < d2 ? H : d2;        // diagonals packed into one output
    int levels = 0;
    for (uint32_t sh = 1; sh < wdt; sh <<= 1) {
        CG_REQUIRE(gk_right[levels] && aligned16(gk_right[levels]));
        levels++;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    const size_t ct2 = (size_t)2 * c->k * c->N;
    const double LB = (double)limb_bytes(c);
    Bump w = bump(c, ws);
    uint64_t *y = w.take<uint64_t>((size_t)2 * c->k * batch);
    // y[u] = x[u] * mask0 (keeps slot 0 of every block)
    const size_t rows = (size_t)batch * 2 * c->k;
    CG_TRY(launch_mulplain(c, s, rows, x, static_cast<const double *>(mask0), 0, 0, StInvU64{y, c->logn},
                           LB * (2.0 * rows + c->k)));
    // pairwise tree inside every group of wdt consecutive units: at level l (shift 2^l)
    // y[j 2^(l+1)] += rotate_right(y[j 2^(l+1) + 2^l], 2^l); rotate right by sh = Galois 3^(N/2 - sh)
    // (the last level leaves one ciphertext per group: straight to the output)
    for (int l = 0; l < levels; l++) {
        const uint32_t sh = 1u << l;
        const size_t stride = (size_t)2 * sh * ct2;
        const bool last = l + 1 == levels;
        CG_TRY(do_rotate(c, s, y + (size_t)sh * ct2, pow3_mod((uint32_t)c->N / 2 - sh, 2u * c->N), gk_right[l], last ? out : y,
                         batch / (2 * sh), 1, w.p, stride, last ? ct2 : stride, y, stride));
    }
    return CG_OK;
}

// One token times `units` plaintext matrices (the decode step's ciphertext-plaintext vector-matrix
// product): rotated copies of the token by a doubling tree, the products with the diagonals summed
// on the way into one inverse transform per unit, then the sum over residue classes modulo d2.
// gk_copies != null: the rotated copies of the token are a series of hoisted rotations of the token
// itself (copy c by 3^c, key gk_copies[c - 1]) instead of the doubling tree over gk_shift
static int cpvm_impl(cg_ctx *c, void *stream, const uint64_t *x, const void *diags, uint32_t units, uint32_t n_diag,
                     uint32_t d2, const void *const *gk_shift, const void *const *gk_copies,
                     const void *const *gk_block, uint64_t *out, void *ws, uint32_t block_w = 0)
{
    CG_REQUIRE(c && ptrs_ok({x, diags, out, ws}) && gk_block && batch_ok(units) && pow2_d(c, d2));
    CG_REQUIRE(n_diag >= 1 && n_diag <= 64 && (n_diag & (n_diag - 1)) == 0 && n_diag <= d2);
    CG_REQUIRE(n_diag == 1 || gk_shift || gk_copies);
    CG_REQUIRE(!overlap(x, 2 * (size_t)c->k * limb_bytes(c), out, 2 * (size_t)c->k * limb_bytes(c) * units));
    if (gk_copies) {
        for (uint32_t cc = 1; cc < n_diag; cc++) CG_REQUIRE(gk_copies[cc - 1] && aligned16(gk_copies[cc - 1]));
    } else {
        int levels = 0;
        for (uint32_t sh = 1; sh < n_diag; sh <<= 1, levels++) CG_REQUIRE(gk_shift[levels] && aligned16(gk_shift[levels]));
    }
    uint32_t gs[20];
    const int nrot = block_generators(c, d2, gs);
    FoldRounds R;
    if (block_w) {
        CG_REQUIRE(fold_rounds(c, gs, nrot, block_w, R) && fold_keys_ok(R, gk_block));
    } else {
        for (int i = 0; i < nrot; i++) CG_REQUIRE(gk_block[i] && aligned16(gk_block[i]));
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    const size_t ct2 = (size_t)2 * c->k * c->N;
    const double LB = (double)limb_bytes(c);
    Bump w = bump(c, ws);
    uint64_t *copies = w.take<uint64_t>((size_t)2 * c->k * n_diag);
    double *f = w.take<double>((size_t)2 * c->k * n_diag);
    uint64_t *xa = w.take<uint64_t>((size_t)2 * c->k * units), *xb = w.take<uint64_t>((size_t)2 * c->k * units);
    // (hoisted: copy 0 is x itself and stays where it is)
    const bool hoisted = gk_copies && n_diag > 1;
    if (!hoisted) CG_TRY(do_copy(c, s, x, ct2, copies, ct2, 1));
    if (hoisted) {
        uint32_t cg[64];
        for (uint32_t cc = 1; cc < n_diag; cc++) cg[cc - 1] = pow3_mod(cc, 2u * c->N);
        CG_TRY(do_rotate_hoisted(c, s, x, ct2, n_diag - 1, cg, gk_copies, copies + ct2, n_diag, 1, w.p));
    } else {
        // copy 2^l + i = copy i rotated left by 2^l
        for (uint32_t sh = 1, l = 0; sh < n_diag; sh <<= 1, l++)
            CG_TRY(do_rotate(c, s, copies, pow3_mod(sh, 2u * c->N), gk_shift[l], copies + (size_t)sh * ct2, sh, 0, w.p));
    }
    const size_t crows = (size_t)n_diag * 2 * c->k, rows = (size_t)units * 2 * c->k;
    const int x_rows = 2 * c->k;
    CG_TRY(launch_fwd(c, s, crows, LdRowsFirst{hoisted ? x : copies, copies + ct2, x_rows, c->k, c->logn}, StF64Red{f, c->logn},
                      KID_FWD_ROWS, LB * 2.0 * crows));
    CG_TRY(launch_inv(c, s, rows, LdInvPlainSum{f, static_cast<const double *>(diags), (int)n_diag, c->logn},
                      StInvU64{xa, c->logn}, KID_INV_MULPLAIN,
                      LB * (crows + (double)units * n_diag * c->k + rows)));
    if (block_w) return fold_chain(c, s, xa, xb, out, R, gk_block, units, w.p);
    return rotate_add_chain(c, s, xa, xb, out, gs, gk_block, nrot, units, w.p);
}
extern "C" int cg_cpvm(cg_ctx *c, void *stream, const uint64_t *x, const void *diags, uint32_t units,
                       uint32_t n_diag, uint32_t d2, const void *const *gk_shift, const void *const *gk_block,
                       uint64_t *out, void *ws)
{
    return cpvm_impl(c, stream, x, diags, units, n_diag, d2, gk_shift, nullptr, gk_block, out, ws);
}
extern "C" int cg_cpvm_hoisted(cg_ctx *c, void *stream, const uint64_t *x, const void *diags, uint32_t units,
                               uint32_t n_diag, uint32_t d2, uint32_t block_round_bits,
                               const void *const *gk_copies, const void *const *gk_block, uint64_t *out, void *ws)
{
    CG_REQUIRE(n_diag == 1 || gk_copies);
    return cpvm_impl(c, stream, x, diags, units, n_diag, d2, nullptr, gk_copies, gk_block, out, ws, block_round_bits);
}

// Every transform-kernel instantiation this context can launch, at a batch below and one above the
// number of compute units (the forward plan depends on it).  Runs with c->dry set: the launch
// helpers look the kernel's occupancy up, record it and return before launching, so the dummy
// addresses are never dereferenced.
static int warm_launch_table(cg_ctx *c)
{
    hipStream_t s = nullptr;
    uint64_t *u = reinterpret_cast<uint64_t *>(uintptr_t(1) << 20);
    double *f = reinterpret_cast<double *>(uintptr_t(1) << 20);
    const double LB = 0.0;
    c->dry_rows = true;
    CG_TRY(do_mul(c, s, u, u, u, 1, 1, f, 0));
    CG_TRY(do_mul(c, s, u, u, u, 2, 2, f, 0));
    CG_TRY(do_mul(c, s, u, u, u, 2, 1, f, 0, 0, 0, nullptr, 2));
    CG_TRY(do_mul(c, s, u, u, u, 2, 2, f, 0, 2, 2, f));
    CG_TRY(do_mul(c, s, u, u, u, 2, 1, f, 0, 2, 2, f, 2));
    CG_TRY(do_keyswitch(c, s, u, 0, 0, f, u, 0, u, 0, 0, 0, 1, f));
    CG_TRY(do_keyswitch(c, s, u, 0, 3, f, u, 0, u, 0, 3, 1, 1, f));
    {
        const uint32_t gs1[1] = {3};
        const void *const keys1[1] = {f};
        CG_TRY(do_rotate_sum(c, s, u, 0, 1, gs1, keys1, u, 0, 1, f));
        CG_TRY(do_rotate_hoisted(c, s, u, 0, 1, gs1, keys1, u, 1, 1, f));
    }
    c->dry_rows = false;
    c->dry_units = true;
    CG_TRY(do_keyswitch(c, s, u, 0, 0, f, u, 0, u, 0, 0, 0, 1, f));
    CG_TRY(do_keyswitch(c, s, u, 0, 3, f, u, 0, u, 0, 3, 1, 1, f));
    {
        const uint32_t gs1[1] = {3};
        const void *const keys1[1] = {f};
        CG_TRY(do_rotate_sum(c, s, u, 0, 1, gs1, keys1, u, 0, 1, f));
    }
    c->dry_units = false;
    for (uint32_t batch : {1u, 4096u}) {
        CG_TRY(do_mul(c, s, u, u, u, batch, 1, f, 0));
        CG_TRY(do_mul(c, s, u, u, u, batch, 1, f, 0, 0, 0, nullptr, 1));
        CG_TRY(do_keyswitch(c, s, u, 0, 0, f, u, 0, u, 0, 0, 0, batch, f));
        CG_TRY(do_keyswitch(c, s, u, 0, 3, f, u, 0, u, 0, 3, 1, batch, f));
        {
            const uint32_t gs1[1] = {3};
            const void *const keys1[1] = {f};
            CG_TRY(do_rotate_hoisted(c, s, u, 0, 1, gs1, keys1, u, 1, batch, f));
            CG_TRY(do_rotate_sum(c, s, u, 0, 1, gs1, keys1, u, 0, batch, f));
        }
        CG_TRY(transform_ext(c, s, MulSrc{nullptr, u, 0, 1, 1, c->logn, 1}, 2 * (size_t)batch, f));
        const size_t rows = (size_t)batch * 2 * c->k;
        const LdRowsU64 ld{u, nullptr, c->k, c->logn};
        CG_TRY(launch_fwd(c, s, rows, ld, StU64{u, c->logn}, KID_FWD_ROWS, LB));
        CG_TRY(launch_fwd(c, s, rows, ld, StF64{f, c->logn}, KID_FWD_ROWS, LB));
        CG_TRY(launch_fwd(c, s, rows, ld, StF64Red{f, c->logn}, KID_FWD_ROWS, LB));
        CG_TRY(launch_fwd(c, s, rows, LdRowsFirst{u, u, 1, c->k, c->logn}, StF64Red{f, c->logn}, KID_FWD_ROWS, LB));
        CG_TRY(launch_fwd(c, s, rows, LdPlain{u, c->logn}, StF64Red{f, c->logn}, KID_FWD_PLAIN, LB));
        CG_TRY(launch_inv(c, s, rows, LdInvU64{u, nullptr, c->k, c->logn}, StInvU64{u, c->logn}, KID_INV_U64, LB));
        const LdInvMulPlain mp{f, f, 1, 1, 0, 0, c->logn};
        CG_TRY(launch_inv(c, s, rows, mp, StInvU64{u, c->logn}, KID_INV_MULPLAIN, LB));
        CG_TRY(launch_mulplain(c, s, rows, u, f, 0, 0, StInvU64{u, c->logn}, LB));
        CG_TRY(launch_mulplain(c, s, rows, u, f, 0, 0, StInvAppend{u, 0, 1, c->logn}, LB));
        CG_TRY(launch_inv(c, s, rows, LdInvPlainSum{f, f, 1, c->logn}, StInvU64{u, c->logn}, KID_INV_MULPLAIN, LB));
    }
    return CG_OK;
}

extern "C" int cg_profile_begin(cg_ctx *c, uint32_t max_launches)
{
    CG_REQUIRE(c && max_launches >= 1 && max_launches <= (1u << 20) && !c->prof_on);
    if (c->prof_cap < max_launches) {
        for (uint32_t i = 0; i < 2 * c->prof_cap; i++) (void)hipEventDestroy(c->prof_ev[i]);
        delete[] c->prof_ev; delete[] c->prof_id; delete[] c->prof_bytes; delete[] c->prof_items;
        c->prof_cap = 0;
        c->prof_ev = new (std::nothrow) hipEvent_t[2 * (size_t)max_launches];
        c->prof_id = new (std::nothrow) uint8_t[max_launches];
        c->prof_bytes = new (std::nothrow) double[max_launches];
        c->prof_items = new (std::nothrow) double[max_launches];
        if (!c->prof_ev || !c->prof_id || !c->prof_bytes || !c->prof_items) return CG_ENOMEM;
        for (uint32_t i = 0; i < 2 * max_launches; i++) CG_HIP(hipEventCreate(&c->prof_ev[i]));
        c->prof_cap = max_launches;
    }
    c->prof_n = 0;
    c->prof_on = true;
    return CG_OK;
}

extern "C" int cg_profile_end(cg_ctx *c, cg_kernel_stat *stats, uint32_t cap, uint32_t *n_out)
{
    CG_REQUIRE(c && stats && n_out && c->prof_on);
    c->prof_on = false;
    cg_kernel_stat acc[KID_COUNT];
    memset(acc, 0, sizeof(acc));
    for (uint32_t i = 0; i < c->prof_n; i++) {
        CG_HIP(hipEventSynchronize(c->prof_ev[2 * i + 1]));
        float ms = 0.f;
        CG_HIP(hipEventElapsedTime(&ms, c->prof_ev[2 * i], c->prof_ev[2 * i + 1]));
        cg_kernel_stat &k = acc[c->prof_id[i]];
        k.launches++;
        k.total_ms += ms;
        k.algo_bytes += c->prof_bytes[i];
        k.work_items += c->prof_items[i];
    }
    uint32_t n = 0;
    for (int id = 0; id < KID_COUNT; id++)
        if (acc[id].launches && n < cap) {
            acc[id].kernel_id = (uint32_t)id;
            stats[n++] = acc[id];
        }
    *n_out = n;
    return CG_OK;
}

extern "C" const char *cg_kernel_name(uint32_t id) { return id < KID_COUNT ? kKernelNames[id] : "?"; }

extern "C" int cg_bench_exchange(cg_ctx *c, void *stream, int kind, uint32_t n_blocks, uint32_t iters, double *out)
{
    CG_REQUIRE(c && ptrs_ok({out}) && (kind == 0 || kind == 1) && n_blocks >= 1 && n_blocks <= (1u << 16));
    return launch_kernel(bench_exchange_kernel, dim3(n_blocks), dim3(1024), static_cast<hipStream_t>(stream), kind,
                         iters, out);
}

extern "C" int cg_bench_modmul(cg_ctx *c, void *stream, int kind, uint32_t n_lanes, uint32_t iters, uint64_t *out)
{
    CG_REQUIRE(c && ptrs_ok({out}) && (kind == 0 || kind == 1) && n_lanes >= 1 && c->pr[0] > (1ull << 49));
    ModI mi{c->pr[0], (uint64_t)((((u128)1) << 100) / c->pr[0])};
    return launch_kernel(bench_modmul_kernel, dim3((n_lanes + PW_THREADS - 1) / PW_THREADS), dim3(PW_THREADS),
                         static_cast<hipStream_t>(stream), kind, n_lanes, iters, out, c->hc.mod[0], mi);
}
