// Internal declarations of libcachemir: modular limb arithmetic for gfx950, context tables
// and kernel launchers.  Not part of the C ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <map>
#include <new>
#include <vector>

#include "../../include/cachemir.h"

typedef uint64_t u64;
typedef unsigned __int128 u128;

// ---- 64-bit modular arithmetic -----------------------------------------------------------
// All moduli are below 2^61 (the lazy sums of the transforms use up to 8 q of a word).  Three multiplier forms are used:
//   Shoup:      constant w with companion wp = floor(w 2^64 / q); result in [0, 2q) (lazy).
//   Montgomery: one operand pre-multiplied by 2^64 mod q; products are accumulated in 128
//               bits and reduced once (REDC), result in [0, q).
struct ModC {
    u64 q;
    u64 qinv;   // q^{-1} mod 2^64
    u64 r2;     // 2^128 mod q
};

__host__ __device__ __forceinline__ u64 mulhi64(u64 a, u64 b) {
#ifdef __HIP_DEVICE_COMPILE__
    return __umul64hi(a, b);
#else
    return (u64)(((u128)a * b) >> 64);
#endif
}

// a*w mod q in [0, 2q) for any a < 2^64
__device__ __forceinline__ u64 mul_shoup_lazy(u64 a, u64 w, u64 wp, u64 q) {
    return a * w - mulhi64(a, wp) * q;
}
__device__ __forceinline__ u64 mul_shoup(u64 a, u64 w, u64 wp, u64 q) {
    u64 r = mul_shoup_lazy(a, w, wp, q);
    return r >= q ? r - q : r;
}
// T 2^-64 mod q in [0, q), for T with (T >> 64) < q
__device__ __forceinline__ u64 redc(u128 T, u64 q, u64 qinv) {
    u64 lo = (u64)T, hi = (u64)(T >> 64);
    u64 t = mulhi64(lo * qinv, q);
    u64 r = hi - t;
    return hi < t ? r + q : r;
}
// a 2^64 mod q
__device__ __forceinline__ u64 to_mont(u64 a, const ModC &m) { return redc((u128)a * m.r2, m.q, m.qinv); }
__device__ __forceinline__ u64 addmod(u64 a, u64 b, u64 q) {
    u64 s = a + b;
    return s >= q ? s - q : s;
}
__device__ __forceinline__ u64 submod(u64 a, u64 b, u64 q) { return a >= b ? a - b : a + q - b; }

// Sum of products d * w with d below 2^50 held as two 25-bit halves (d = d0 + 2^25 d1) and w any 64-bit word: four
// 32 x 32 -> 64-bit multiply-adds into four accumulators that cannot overflow for up to 16 terms (each term is below
// 2^57), so a product costs four instructions and no carry chain; the accumulators are combined once per sum.  The
// generic form (64 x 64 -> 128 with carries, about ten instructions) stays for the 60-bit moduli.
struct Acc50 {
    u64 t00 = 0, t01 = 0, t10 = 0, t11 = 0;
    __device__ __forceinline__ void mac(unsigned d0, unsigned d1, u64 w) {
        const unsigned w0 = (unsigned)w, w1 = (unsigned)(w >> 32);
        t00 += (u64)d0 * w0, t01 += (u64)d0 * w1, t10 += (u64)d1 * w0, t11 += (u64)d1 * w1;
    }
    __device__ __forceinline__ u128 total() const {
        return (u128)t00 + ((u128)t01 << 32) + ((u128)t10 << 25) + ((u128)t11 << 57);
    }
};
#define LOW25 0x1FFFFFFu
#define LOW30 0x3FFFFFFFu

// Position i of the evaluation order holds the value at psi^(2 brev(i) + 1); the Galois map
// X -> X^g moves the value at exponent e*g to exponent e: out[i] = in[perm_src(i, g)].  It maps
// aligned blocks of 2^k positions onto aligned blocks (and i^1 to src^1).
__device__ __forceinline__ unsigned perm_src(unsigned i, unsigned g, int logn) {
    unsigned e = 2u * (__brev(i) >> (32 - logn)) + 1u;
    unsigned s = (e * g) & ((2u << logn) - 1u);
    return __brev((s - 1u) >> 1) >> (32 - logn);
}

// A multiplier w of the integer butterflies under a modulus q = 2^b - c from 2^50 on, cut up so that its product with a = a0 + 2^32 a1
// is two sums of two 32 x 32-bit products: w = w0 + 2^30 (w1 2^(b-61)) and w 2^32 mod q = v0 + 2^30 (v1 2^(b-61)).  The upper parts
// are scaled by 2^(61-b), whatever b, so that the weight 2^(b+1) of the upper sum's upper word is 2 c (IntArith::mul).
struct IntTw {
    unsigned w0, w1, v0, v1;
};

// modulus as doubles for the FP64 butterflies (moduli below 2^50 only; q = 0 otherwise)
struct FpQ {
    double q, qinv;       // modulus and 1/q as doubles; q = 0 where the modulus is too large for the FP64 paths
    double rinv, rinvq;   // 2^-64 mod q and that over q: takes a product with a multiplier-form operand back
};

// ---- context -----------------------------------------------------------------------------
#define CM_MAX_LIMBS 64
#define CM_MAX_DIGITS 16
#define CM_GAUSS_K 19
#define CM_KS_BATCH 8      // hoisted rotations whose ModDown runs as one batch
#define CM_MASK_BATCH 32   // masked products of a cache append in one batch, at most (rescale_masked_batch)
#define CM_NTT_MAX_LIMBS 1024

struct ConvTable {            // fast base conversion src -> dst (all indices into the modulus list)
    int ns = 0, nt = 0;
    std::vector<u64> inv_hat;     // [ns]   (hat_m^{-1} mod q_m), plain
    std::vector<u64> inv_hat_sh;  // [ns]   Shoup companion
    std::vector<u64> hat_mont;    // [ns*nt] (hat_m mod r) 2^64 mod r
    std::vector<u64> hat;         // [ns*nt] hat_m mod r
    std::vector<int> src, dst;
};

// The same table in the form the conversion kernel reads (one per digit / per direction).
#define CONV_MAX_SRC 8
#define CONV_MAX_DST 64
// split: how a product y_m * weight is formed without carry chains (all source moduli below 2^50; source moduli below 2^60
// and target moduli below 2^50; otherwise plain 128-bit sums).  Rows past ns are zero (a zero inverse, zero weights, input
// row 0), so that a kernel may run over a fixed number of sources.
enum { CONV_SPLIT_25 = 0, CONV_SPLIT_30 = 1, CONV_SPLIT_NONE = 2 };
// A weight w of the conversion to q = 2^b - c and v = w 2^s mod q, s = 25 or 30 the bits of the lower part of a y_m = y0 + 2^s y1 (by
// `split`), each as x0 + 2^t x1.  Below 2^50 t = ceil(b / 2), from there 30; the upper parts are scaled up by 2^z so that the upper word
// of h = sum y0 w1 + y1 v1 has the weight 2^(b+3) = 8 c (z = 29 - (b - t)) or 2^(b+1) = 2 c (z = 61 - b):
//   sum y_m w_m = l + mlo (h mod 2^32) + mhi (h >> 32)  (mod q),   l = sum y0 w0 + y1 v0,  mlo = 2^(t-z),  mhi = 8 c or 2 c.
// With up to nine terms below 2^60 (target below 2^50) or nine below 2^50 or four below 2^60 (others) nothing passes 2^64.
struct ConvCut {
    unsigned w0, w1, v0, v1;
};
// one target modulus: everything the conversion to it reads, in one record
struct ConvTarget {
    int mod, row;                 // modulus index, output row
    double qd;                    // the modulus as a double, 0 from 2^50 on (integer arithmetic)
    double w[CONV_MAX_SRC];       // hat_m mod q (exact for moduli below 2^50)
    u64 q, qinv;                  // modulus, q^{-1} mod 2^64
    u64 wm[CONV_MAX_SRC];         // hat_m mod q in multiplier form
    double wl;                    // the same of the weight of a folded last limb (ConvDev::fold): P mod q
    u64 wlm;
    // the same weights cut up (ConvDev::near); q = 2^b - c, cb = b - 32, twice: b < 49 (a second fold)
    unsigned c, cb, mlo, mhi, twice;
    ConvCut cut[CONV_MAX_SRC], cutl;
};
struct ConvDev {
    int ns, nt, split;
    int near;                     // all targets are close below a power of two and the sums of the cut weights fit
    int in_rows[CONV_MAX_SRC];
    // a single source whose inverse transform is part of the conversion (ConvBatch::inv): its modulus index, and n^-1 inv_hat, the last
    // factor of that transform with its own (below 2^50 as a double, above cut up)
    int src_mod;
    double inv_hat_nd;
    IntTw inv_hat_n;
    u64 inv_hat[CONV_MAX_SRC], inv_hat_sh[CONV_MAX_SRC], src_q[CONV_MAX_SRC];
    double src_qd[CONV_MAX_SRC], inv_hat_d[CONV_MAX_SRC], inv_hat_dq[CONV_MAX_SRC];   // q_m, inv_hat_m, inv_hat_m / q_m as doubles
    ConvTarget t[CONV_MAX_DST];
    // ModDown and rescale in one (ks_drop): one more source, the limb x of row `row` under q_level, enters as
    // (x - sum_m y_m hat_m) P^-1 mod q_level with the weight P
    struct {
        int row;
        ConvTarget t;             // the conversion to q_level
        u64 pinv, pinv_sh;        // P^{-1} mod q_level
    } fold;
};

// per-kernel-family timing with HIP events on the launching stream (off unless enabled)
struct ProfState {
    bool on = false;
    std::vector<hipEvent_t> pool;
    struct Rec { int fam; double units; size_t e0; };
    std::vector<Rec> recs;
};

struct cm_ctx {
    cm_params prm;
    ProfState prof;
    int n, logn, L, K, alpha, nmod;      // nmod = L+1+K
    std::vector<u64> mod;                 // host copy of moduli
    std::vector<u64> psi;
    // device tables, indexed by modulus index
    ModC *d_modc = nullptr;               // [nmod]
    u64 *d_pmont = nullptr;               // [L+1] P = p_0 .. p_{K-1} mod q_i, multiplier (Montgomery) form
    u64 *d_ubound = nullptr;              // [nmod] q * floor(2^64 / q): uniform draws at or above it are rejected
    // twiddles psi^brev(i) of the moduli from 2^50 on [nmod][n], forward and inverse, and n^{-1} [nmod]
    IntTw *d_tw = nullptr, *d_itw = nullptr, *d_ninv = nullptr;
    // the same as doubles (w and w/q) for the limbs whose modulus is below 2^50
    FpQ *d_fpq = nullptr;                       // [nmod] (q, 1/q), q = 0 for larger moduli
    double *d_twd = nullptr, *d_twqd = nullptr, *d_itwd = nullptr, *d_itwqd = nullptr;
    double *d_ninvd = nullptr, *d_ninvqd = nullptr;
    std::vector<ModC> modc;
    // per-level tables (built lazily, kept): ModUp per digit, ModDown, rescale constants
    std::map<int, std::vector<ConvTable>> modup;   // level -> digit tables
    std::map<int, ConvTable> moddown;              // level -> P -> q_0..q_level
    std::map<int, u64 *> pinv;                     // level -> [level+1][2]: P^{-1} mod q_i, Shoup
    std::map<int, u64 *> qlinv;                    // level -> [level][2]: q_level^{-1} mod q_i, Shoup
    u64 *d_cdt = nullptr;                          // Gaussian table [CM_GAUSS_K]
    u64 cdt[CM_GAUSS_K];
    int lazy_terms;                                // products that may be summed before one REDC
    // options (cm_ctx_set_option)
    bool evk_stored_a = false;     // evaluation keys carry both halves; the inner products read the uniform half
    bool two_step_masks = false;   // cache appends multiply, store and rescale instead of fusing the product into the rescale
    // scratch arena
    u64 *arena = nullptr;
    size_t arena_words = 0;
    int *d_idx = nullptr;                          // 0, 1, 2, ...: modulus index lists of consecutive limbs
    int *d_idx_stage = nullptr;                    // [CM_NTT_MAX_LIMBS] staging of a caller's modulus index list (cm_ntt)
    // encode tables (host)
    std::vector<int> slot_pos;
    std::vector<double> tw_re, tw_im;              // omega^k
};

struct cm_sk {
    std::vector<int8_t> coeffs;
    u64 *d_ntt = nullptr;          // [nmod][n], Montgomery form, evaluation domain
    u64 noise = 0;                 // XORed into the public seed of a call to key its error streams
};

struct EvkEntry {
    u64 *d = nullptr;              // b halves [digits][nmod][n] (multiplier form, evaluation domain), then the
                                   // [digits][nmod] generator keys of the streams of the a halves (padded to an even
                                   // count), then -- stored_a only -- the a halves [digits][nmod][n] in multiplier form
};
struct cm_evk {
    int digits;
    bool stored_a = false;         // the option the set was generated under
    u64 seed = 0;                  // the (public) seed every key of the set was generated from
    std::map<u64, EvkEntry> keys;  // Galois element (0 = relinearisation)
};
// word offset of the stored a halves inside a key
inline size_t evk_a_offset(const cm_ctx *ctx) {
    const size_t digits = (size_t)(ctx->L + ctx->alpha) / ctx->alpha, nm = (size_t)ctx->nmod;
    return digits * nm * ctx->n + ((digits * nm + 1) & ~(size_t)1);
}

#define HIPCHK(x)                                  \
    do {                                           \
        hipError_t e_ = (x);                       \
        if (e_ != hipSuccess) {                    \
            cm_set_hip_error((int)e_);             \
            return CM_E_HIP;                       \
        }                                          \
    } while (0)
// Kernel launches report a bad configuration only through the runtime's last-error slot: the hot
// entry points end with this check (no synchronisation).
#define RETURN_LAUNCH_STATUS()                     \
    do {                                           \
        hipError_t e_ = hipPeekAtLastError();      \
        if (e_ != hipSuccess) {                    \
            cm_set_hip_error((int)e_);             \
            return CM_E_HIP;                       \
        }                                          \
        return CM_OK;                              \
    } while (0)
#define CMCHK(x)                \
    do {                        \
        cm_status s_ = (x);     \
        if (s_ != CM_OK) return s_; \
    } while (0)

void cm_set_hip_error(int e);
// Every extern "C" body that can reach an allocation (std::vector, std::map, new) sits between these: no C++
// exception crosses the boundary.
#define CM_TRY try {
#define CM_CATCH                                        \
    }                                                   \
    catch (const std::bad_alloc &) { return CM_E_NOMEM; } \
    catch (...) { return CM_E_INVAL; }

struct Prof {
    cm_ctx *c;
    hipStream_t st;
    size_t e0;
    bool live;
    Prof(cm_ctx *ctx, int fam, double units, hipStream_t st);
    ~Prof();
};

// ---- host helpers (context.hip) ------------------------------------------------------------
u64 h_mulmod(u64 a, u64 b, u64 q);
u64 h_powmod(u64 b, u64 e, u64 q);
u64 h_invmod(u64 a, u64 q);
u64 h_shoup(u64 w, u64 q);
IntTw h_int_tw(u64 w, u64 q);
ConvCut conv_cut(u64 q, u64 w, int s);         // of a weight w for a target q
u64 galois_of_step(const cm_ctx *ctx, int step);
const std::vector<ConvTable> &get_modup(cm_ctx *ctx, int level);
const ConvTable &get_moddown(cm_ctx *ctx, int level);
const u64 *get_pinv(cm_ctx *ctx, int level);
const u64 *get_qlinv(cm_ctx *ctx, int level);
std::vector<std::vector<int>> digits_at(const cm_ctx *ctx, int level);

// ---- kernel launchers ----------------------------------------------------------------------
// ntt.hip: limbs of n words each, limb i under modulus d_mod_idx[i] (device int array)
void launch_ntt(cm_ctx *ctx, u64 *data, const int *d_mod_idx, int limbs, bool inverse, hipStream_t st);
// convenience: limbs use consecutive modulus indices first, first+1, ...
void launch_ntt_range(cm_ctx *ctx, u64 *data, int first_mod, int limbs, bool inverse, hipStream_t st);
const int *iota_idx(cm_ctx *ctx);   // device array 0,1,2,...,CM_MAX_LIMBS-1
