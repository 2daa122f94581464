// Batched negacyclic NTT / inverse NTT over RNS limbs for gfx950.
//
// Transform: a(X) in Z_q[X]/(X^n+1)  ->  values a(psi^(2 brev(i)+1)) at position i (bit-reversed
// evaluation order), the merged-twiddle Cooley-Tukey / Gentleman-Sande pair.
//
// Decomposition for the 64-wide machine: n = 256 * n2.  A workgroup of 256 lanes owns 4096
// words; every lane keeps 16 of them in registers and runs four butterfly stages there
// (radix 16), then the workgroup transposes through LDS and runs four more.
//   column kernel : stages 0..7, a tile of 256 rows x 16 adjacent columns (rows n2 apart)
//   row kernel    : the remaining log2(n2) stages on contiguous blocks of n2 words
// so a limb makes two round trips to HBM for n = 65536.  For n = 4096 the limb is one tile and both parts run in one kernel.
//
// Two butterfly arithmetics, chosen per limb (uniform per workgroup):
//   IntArith : lazy butterflies on u64 (moduli 2^b - c, 50 < b <= 61); about 18 VALU instructions per butterfly with its share
//              of the folds.
//   FpArith  : for moduli below 2^50, residues held as exact integers in doubles.  FP64 FMA
//              issues at full rate here, and a modular product is 6 instructions:
//                  h = y*w; l = fma(y, w, -h)            (exact product h + l)
//                  c = rint(y * (w/q)); r = fma(-c, q, h) + l
//              exact because |h - c q| < 2^53 whenever |y| < 8 q; r = y w (mod q).
//              Values stay signed and lazy (below 8 q = 2^53); a forward butterfly is 8 instructions, an
//              inverse one 11 (see FpArith).  Between the two kernels of a
//              transform the words in memory are raw doubles; at rest they are u64 in [0, q).
// Both give bit-identical results (all steps are exact integer arithmetic).
#include "kernels.h"

#define NTT_THREADS 256

// The start of the largest kernels, 14 to 52 KiB of code that every short launch fetches anew: where they lie in the code object moves the
// calls made of such launches (rotary embedding at level 3 69.6 and 70.2 us with the same instructions 1 KiB further on; 69.2 so).
#define CODE_ALIGN __attribute__((aligned(4096)))

struct NttTables {
    const ModC *modc;
    const IntTw *tw;              // [nmod][n] integer twiddles
    const double *twd, *twqd;     // [nmod][n] the same twiddles as doubles, and w/q
    const IntTw *ninv;            // [nmod] n^{-1} (inverse only)
    const double *ninvd, *ninvqd;
    const FpQ *fpq;               // [nmod] q and 1/q as doubles; q = 0 where the limb must use IntArith
    // Large launches (256 limbs and more) read with non-temporal loads: their input was written long before and is read
    // once.  Small launches find theirs in the caches and read plainly (a single key switch is 3 % slower otherwise).
    // A limb is read again only by a later kernel.  Large launches write with non-temporal stores (after hundreds of MiB of
    // other limbs have gone by; 1 % off the transforms of a step against plain stores), small ones at agent scope, through to
    // memory at once instead of when the L2 evicts or a kernel ends: plain transforms of 24 to 255 limbs take 5 to 40 % less.  Against
    // non-temporal stores: ciphertext product at level 13 158.5 -> 154.2 us, rotary embedding at level 3 138.0 -> 134.9, 4096 x 4096
    // product at level 4 1154 -> 1140; for large launches agent scope is 2 to 5 % slower (attention, product at level 23), plain stores
    // 1 to 4 %.  The column pass of a conversion draws the line at CCF_NT limbs.
    int large;
};

// element idx of a uniform array by a 32-bit byte offset (one register and the scalar base, no 64-bit address arithmetic)
template <class T>
__device__ __forceinline__ T *word_at(T *base, unsigned idx) {
    return (T *)((char *)base + idx * (unsigned)sizeof(T));
}
template <class T>
__device__ __forceinline__ const T *word_at(const T *base, unsigned idx) {
    return (const T *)((const char *)base + idx * (unsigned)sizeof(T));
}

// ---- integer arithmetic --------------------------------------------------------------------------
// Moduli q = 2^b - c, 51 <= b <= 61; the primes of a context are the first ones below 2^b in steps of 2n, at most 64 of them, so c
// is below 2^28.  Residues stay lazy: a value is only kept below 2^64, i.e. below 16 q (8 q for 61-bit moduli, `tight`).
// A product with a twiddle uses what q looks like instead of a quotient.  With the twiddle cut up as IntTw says and any a =
// a0 + 2^32 a1 below 2^64,
//   l = a0 w0 + a1 v0 < 2^63,  h = a0 w1 + a1 v1 < 2^64,  a w = l + 2^(b-31) h  (mod q)  =  l + 2^(b-31) (h mod 2^32) + 2^(b+1) (h >> 32)
// and 2^(b+1) = 2 c: six multiply-adds without a carry, their sum below 2^63 + 2^(b+1) + 2^33 c < 2^64.  A fold, v = (v mod 2^b) +
// (v >> b) c, three instructions, leaves less than 2^b + 2^13 c < q + q / 512.  Nine instructions; a product with a Shoup twiddle
// (quotient from three of its four partial products, below 4 q) took thirteen and moves to zero-extend its halves, a butterfly of
// it 30 with its share of the folds, now 18.  The passes over a few limbs and the conversions wait more than they multiply, so the calls
// gain less: 64 x 64 product at n = 4096 449 -> 422 us, rotary embedding at level 3 76.1 -> 72.2, ciphertext product at level 13 153 -> 148,
// query times K at level 12 16570 -> 16170, decode-step attention at level 3 3490 -> 3410.
// Additions are not reduced; forward, all values are folded after every fourth stage (tight: second), inverse, the sums after every
// second (tight: each).  Bounds in units of q (+ 1/512 a product):
//   forward  4 (input) or 1 -> + 2 a stage -> at most 12, folded to 1; tight: 4 -> 8, folded
//   inverse  2 -> 4 -> 8 (sums), folded to 1; products 1; tight: 2 -> 4, folded
struct IntArith {
    typedef u64 T;
    u64 q;
    unsigned c, bs, mask, up;     // 2^b - q, b - 32, low bits of the upper word, 2^(b-31)
    bool tight;                   // 8 q is the most a word holds
    const IntTw *w;
    IntTw ni;
    __device__ __forceinline__ void init(const NttTables &t, int mi, int n) {
        q = t.modc[mi].q;
        bs = 32 - __clz((unsigned)(q >> 32));
        c = (unsigned)((1ULL << (bs + 32)) - q), mask = (1u << bs) - 1u, up = 2u << bs, tight = bs > 28;
        w = t.tw + (size_t)mi * n;
        ni = IntTw{0, 0, 0, 0};
        if (t.ninv) ni = t.ninv[mi];
    }
    __device__ __forceinline__ T from_rest(u64 raw) const { return raw; }     // inverse: below 2q
    __device__ __forceinline__ T from_lazy(u64 raw) const { return raw; }     // forward: below 4q
    __device__ __forceinline__ T from_mid(u64 raw) const { return raw; }
    __device__ __forceinline__ u64 to_mid(T v) const { return v; }
    typedef IntTw W;
    typedef uint4 Word;                                                       // one 16-byte load
    __device__ __forceinline__ Word word(unsigned idx) const { return *word_at(reinterpret_cast<const uint4 *>(w), idx); }
    __device__ __forceinline__ void pair(const Word &x, W &a, W &) const { a = IntTw{x.x, x.y, x.z, x.w}; }
    __device__ __forceinline__ u64 mul(u64 a, const IntTw &x) const {         // a x mod q, below q + q / 512
        const unsigned a0 = (unsigned)a, a1 = (unsigned)(a >> 32);
        const u64 l = (u64)a0 * x.w0 + (u64)a1 * x.v0, h = (u64)a0 * x.w1 + (u64)a1 * x.v1;
        return fold(l + (u64)(unsigned)h * up + (u64)(unsigned)(h >> 32) * (2 * c));
    }
    __device__ __forceinline__ u64 fold(u64 v) const {
        const unsigned hi = (unsigned)(v >> 32);
        return (u64)(hi >> bs) * c + (((u64)(hi & mask) << 32) | (unsigned)v);
    }
    __device__ __forceinline__ void ct(T &X, T &Y, const W &a, const W &) const {
        const u64 t = mul(Y, a), x = X;
        X = x + t;
        Y = (x + 2 * q) - t;
    }
    __device__ __forceinline__ void gs(T &X, T &Y, const W &a, const W &) const {
        const u64 d = (X + 4 * q) - Y;
        X = X + Y;
        Y = mul(d, a);
    }
    // stage s of the transform is done on all the lane's values
    template <int NV>
    __device__ __forceinline__ void after_fwd(int s, T (&v)[NV]) const {
        if ((s & 3) == 3 || ((s & 1) && tight)) {
#pragma unroll
            for (int k = 0; k < NV; k++) v[k] = fold(v[k]);
        }
    }
    // stage s (the last one first): the sums sit where bit `half` of the index is clear
    template <int NV>
    __device__ __forceinline__ void after_inv(int s, int half, T (&v)[NV]) const {
        if (!(s & 1) || tight) {
#pragma unroll
            for (int k = 0; k < NV; k++)
                if (!(k & half)) v[k] = fold(v[k]);
        }
    }
    __device__ __forceinline__ u64 to_rest_fwd(T v) const { return v >= q ? v - q : v; }
    __device__ __forceinline__ u64 to_tail(T v) const { return to_rest_fwd(v); }
    // (u - conv) pinv (+ a) (+ c), and (u pt - conv) pinv (+ c) with pt in multiplier form
    struct Tail {
        u64 pi, pis, qinv;
        __device__ __forceinline__ Tail(const IntArith &, const NttTables &t, int mi, u64 p, u64 ps) : pi(p), pis(ps), qinv(t.modc[mi].qinv) {}
        // (u - conv) pinv + (a + c) ainv
        __device__ __forceinline__ u64 drop(const IntArith &ar, u64 u, u64 conv, u64 a, u64 c, u64 ai, u64 ais) const {
            return addmod(mul_shoup(submod(u, conv, ar.q), pi, pis, ar.q), mul_shoup(a + c, ai, ais, ar.q), ar.q);
        }
        __device__ __forceinline__ u64 plain(const IntArith &ar, u64 u, u64 conv, bool has_a, u64 a, bool has_c, u64 c) const {
            u64 x = mul_shoup(submod(u, conv, ar.q), pi, pis, ar.q);
            if (has_a) x = addmod(x, a, ar.q);
            if (has_c) x = addmod(x, c, ar.q);
            return x;
        }
        __device__ __forceinline__ u64 masked(const IntArith &ar, u64 u, u64 pt, u64 conv, bool has_c, u64 c) const {
            return plain(ar, redc((u128)u * pt, ar.q, qinv), conv, false, 0, has_c, c);
        }
    };
    __device__ __forceinline__ u64 to_rest_inv(T v) const { return to_rest_fwd(mul(v, ni)); }
};

// ---- FP64 arithmetic for moduli below 2^50 -----------------------------------------------------------
#define TWO52 4503599627370496.0
struct FpArith {
    typedef double T;
    double q, qinv, ni, niq;
    const double *w, *wq;
    __device__ __forceinline__ void init(const NttTables &t, int mi, int n) {
        q = t.fpq[mi].q, qinv = t.fpq[mi].qinv;
        w = t.twd + (size_t)mi * n, wq = t.twqd + (size_t)mi * n;
        ni = niq = 0.0;
        if (t.ninvd) ni = t.ninvd[mi], niq = t.ninvqd[mi];
    }
    __device__ __forceinline__ double mulmod(double y, double a, double aq) const {
        double h = y * a;
        double l = __builtin_fma(y, a, -h);
        double c = __builtin_rint(y * aq);
        return __builtin_fma(-c, q, h) + l;
    }
    __device__ __forceinline__ double norm(double x) const { return __builtin_fma(-__builtin_rint(x * qinv), q, x); }
    __device__ __forceinline__ T from_rest(u64 raw) const {                                     // below 2^52, i.e. 4q
        return __longlong_as_double((long long)(raw | 0x4330000000000000ULL)) - TWO52;
    }
    // What comes into a forward transform need not be reduced (a caller's words, a rescale's last limb under another
    // modulus): brought to q / 2 here, since four stages from 4q would pass 2^53 (three instructions of about 90 a word).
    __device__ __forceinline__ T from_lazy(u64 raw) const { return norm(from_rest(raw)); }
    __device__ __forceinline__ T from_mid(u64 raw) const { return __longlong_as_double((long long)raw); }
    __device__ __forceinline__ u64 to_mid(T v) const { return (u64)__double_as_longlong(v); }
    typedef double W;
    typedef double Word;
    __device__ __forceinline__ Word word(unsigned idx) const { return *word_at(w, idx); }
    __device__ __forceinline__ void pair(Word x, W &a, W &b) const { a = x, b = x * qinv; }
    // Products: |r| <= (1/2 + 3/8 B) q for |y| <= B q (the quotient comes from three roundings of a value below B 2^50).
    // Forward: nothing is renormalised inside four stages; from B = 1 the values grow to 1.88, 3.08, 4.74, 7.02 q, below the
    // 2^53 = 8 q up to which integers are exact, and are brought back to q / 2 after every fourth stage (3 instructions per
    // word and four stages instead of 3 per butterfly).
    // Inverse: sums double, so each is renormalised where it is formed.
    template <int NV>
    __device__ __forceinline__ void after_fwd(int s, T (&v)[NV]) const {
        if ((s & 3) == 3) {
#pragma unroll
            for (int k = 0; k < NV; k++) v[k] = norm(v[k]);
        }
    }
    template <int NV>
    __device__ __forceinline__ void after_inv(int, int, T (&)[NV]) const {}
    __device__ __forceinline__ void ct(T &X, T &Y, W a, W b) const {
        const double x = X, r = mulmod(Y, a, b);
        X = x + r;
        Y = x - r;
    }
    __device__ __forceinline__ void gs(T &X, T &Y, W a, W b) const {
        double s = X + Y, d = X - Y;
        X = norm(s);
        Y = mulmod(d, a, b);
    }
    // |v| < q -> [0, q): q is added under the sign mask
    __device__ __forceinline__ u64 lift(double v) const {
        const int m = __double2hiint(v) >> 31;
        const double a = __hiloint2double(__double2hiint(q) & m, __double2loint(q) & m);
        return (u64)__double_as_longlong((v + a) + TWO52) & 0x000FFFFFFFFFFFFFULL;
    }
    __device__ __forceinline__ u64 canon(double v) const { return lift(norm(v)); }       // |v| < 2^53 -> [0, q)
    __device__ __forceinline__ u64 to_rest_fwd(T v) const { return lift(v); }           // after the last stage's norm
    __device__ __forceinline__ u64 to_tail(T v) const { return to_mid(v); }
    // The tails in FP64: |conv| <= q / 2, so |u - conv| <= 1.5 q, its product at most 1.07 q, and the sum of four terms
    // below 5 q before the one reduction at the end.
    struct Tail {
        double pi, piq, rp, rpq;
        __device__ __forceinline__ Tail(const FpArith &ar, const NttTables &t, int mi, u64 p, u64) {
            pi = (double)p, piq = pi * ar.qinv;
            rp = ar.mulmod(pi, t.fpq[mi].rinv, t.fpq[mi].rinvq), rpq = rp * ar.qinv;         // 2^-64 pinv
        }
        __device__ __forceinline__ u64 plain(const FpArith &ar, u64 u, u64 conv, bool has_a, u64 a, bool has_c, u64 c) const {
            double x = ar.mulmod(ar.from_rest(u) - ar.from_mid(conv), pi, piq);
            if (has_a) x += ar.from_rest(a);
            if (has_c) x += ar.from_rest(c);
            return ar.canon(x);
        }
        __device__ __forceinline__ u64 drop(const FpArith &ar, u64 u, u64 conv, u64 a, u64 c, u64 ai, u64) const {
            const double w = (double)ai;
            return ar.canon(ar.mulmod(ar.from_rest(u) - ar.from_mid(conv), pi, piq) +
                            ar.mulmod(ar.from_rest(a) + ar.from_rest(c), w, w * ar.qinv));
        }
        __device__ __forceinline__ u64 masked(const FpArith &ar, u64 u, u64 pt, u64 conv, bool has_c, u64 c) const {
            const double a = ar.from_rest(pt);
            double x = ar.mulmod(ar.mulmod(ar.from_rest(u), a, a * ar.qinv), rp, rpq) - ar.mulmod(ar.from_mid(conv), pi, piq);
            if (has_c) x += ar.from_rest(c);
            return ar.canon(x);
        }
    };
    __device__ __forceinline__ u64 to_rest_inv(T v) const { return canon(mulmod(v, ni, niq)); }
};

// Twiddle providers for four stages starting at stage s0 with base0 = 2^s0 + (block index):
// stage s0 + a, group g uses table entry (base0 << a) + g.
// Both arithmetics read all fifteen entries up front (one exposure to memory latency instead of one per stage, and the
// loads overlap the data loads or the LDS exchange in front of them).  Integer limbs read a multiplier cut up as
// IntTw, one 16-byte word; FP64 limbs take the second factor w/q as w * (1/q), one multiplication instead
// of a second table: the quotient estimate may then be off by one more unit, the product stays exact
// (|r| <= (1/2 + 3/8 B) q for |y| <= B q, see FpArith).
template <class A, int ST>                      // ST stages
struct Tw {
    const A &ar;
    typename A::Word w[(1 << ST) - 1];
    __device__ __forceinline__ Tw(const A &a_, unsigned b0) : ar(a_) {
#pragma unroll
        for (int a = 0; a < ST; a++)
#pragma unroll
            for (int g = 0; g < (1 << a); g++) w[(1 << a) - 1 + g] = ar.word((b0 << a) + g);
    }
    __device__ __forceinline__ void get(int a, int g, typename A::W &w0, typename A::W &w1) const { ar.pair(w[(1 << a) - 1 + g], w0, w1); }
};
template <class A>
using TableTw = Tw<A, 4>;
// The same entries computed from ONE table word (FP64 limbs): with T_a = tw[base0 << a],
//   T_2 = T_3^2, T_1 = T_2^2, T_0 = T_1^2      (the exponent brev(base0) >> a doubles each time)
//   tw[(base0 << a) + g] = T_a * tw[g]          (the low bits g reverse into the top of the exponent)
// which removes almost all twiddle traffic of the last four stages, where every lane has its own 15.
struct GenTw {
    const FpArith &ar;
    double T[4];
    __device__ __forceinline__ GenTw(const FpArith &a_, u64 base0) : ar(a_) {
        T[3] = ar.w[base0 << 3];
        T[2] = ar.mulmod(T[3], T[3], T[3] * ar.qinv);
        T[1] = ar.mulmod(T[2], T[2], T[2] * ar.qinv);
        T[0] = ar.mulmod(T[1], T[1], T[1] * ar.qinv);
    }
    __device__ __forceinline__ void get(int a, int g, double &w0, double &w1) const {
        w0 = g ? ar.mulmod(T[a], ar.w[g], ar.wq[g]) : T[a];
        w1 = w0 * ar.qinv;
    }
};

// ST forward stages, the first of them stage S0 of the transform, on 2^ST register values whose index is the local position
// inside one butterfly block of the first of these stages.
template <int ST, int S0, class A, class TW>
__device__ __forceinline__ void radix_fwd(typename A::T (&v)[1 << ST], const A &ar, const TW &tw) {
#pragma unroll
    for (int a = 0; a < ST; a++) {
        const int half = (1 << ST) >> (a + 1);
#pragma unroll
        for (int g = 0; g < (1 << a); g++) {
            typename A::W w0, w1;
            tw.get(a, g, w0, w1);
#pragma unroll
            for (int j = 0; j < half; j++) {
                const int k = g * 2 * half + j;
                ar.ct(v[k], v[k + half], w0, w1);
            }
        }
        ar.after_fwd(S0 + a, v);
    }
}
template <class A, class TW>
__device__ __forceinline__ void radix16_fwd_tw(typename A::T (&v)[16], const A &ar, const TW &tw) {
    radix_fwd<4, 0>(v, ar, tw);
}
// The inverse of the above (stages in the opposite order).
template <int ST, int S0, class A, class TW>
__device__ __forceinline__ void radix_inv(typename A::T (&v)[1 << ST], const A &ar, const TW &tw) {
#pragma unroll
    for (int a = ST - 1; a >= 0; a--) {
        const int half = (1 << ST) >> (a + 1);
#pragma unroll
        for (int g = 0; g < (1 << a); g++) {
            typename A::W w0, w1;
            tw.get(a, g, w0, w1);
#pragma unroll
            for (int j = 0; j < half; j++) {
                const int k = g * 2 * half + j;
                ar.gs(v[k], v[k + half], w0, w1);
            }
        }
        ar.after_inv(S0 + a, half, v);
    }
}
template <class A, class TW>
__device__ __forceinline__ void radix16_inv_tw(typename A::T (&v)[16], const A &ar, const TW &tw) {
    radix_inv<4, 0>(v, ar, tw);
}
// last four stages of the row pass: generated twiddles for FP64 limbs, table for the others
__device__ __forceinline__ void radix16_fwd_last(double (&v)[16], const FpArith &ar, u64 base0) {
    radix16_fwd_tw(v, ar, GenTw(ar, base0));
}
__device__ __forceinline__ void radix16_fwd_last(u64 (&v)[16], const IntArith &ar, u64 base0) {
    radix16_fwd_tw(v, ar, TableTw<IntArith>(ar, base0));
}
__device__ __forceinline__ void radix16_inv_last(double (&v)[16], const FpArith &ar, u64 base0) {
    radix16_inv_tw(v, ar, GenTw(ar, base0));
}
__device__ __forceinline__ void radix16_inv_last(u64 (&v)[16], const IntArith &ar, u64 base0) {
    radix16_inv_tw(v, ar, TableTw<IntArith>(ar, base0));
}

// LARGE: the same as NttTables::large, at compile time for the stores (with both kinds behind a branch the passes of 256 limbs and more
// took 1 to 3 % longer: 512 limbs under 58-bit primes 249 us inverse, 241 so; 1008 under 50-bit ones 438 and 431).  Not for the loads:
// without the branch 1008 limbs take 7 % less and 256 to 512 up to 7 % more.
__device__ __forceinline__ void ntt_store(int large, u64 *p, u64 v) {
    if (large) __builtin_nontemporal_store(v, p);
    else __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// the masked products of a cache append read the cached ciphertext they add to and write it back past the caches (the
// cache is gigabytes; 3 % off an append)
#define TAIL_LD(ptr) __builtin_nontemporal_load(ptr)
#define TAIL_ST(ptr, val) __builtin_nontemporal_store((u64)(val), (ptr))
// LDS index with one pad word per 16 so that lanes reading words 16 apart hit distinct banks
__device__ __forceinline__ int pad(int e) { return e + (e >> 4); }
#define LDS_WORDS (4096 + 256)

// ---- column passes: stages 0..7; tile = rows 0..255 of 16 adjacent columns ---------------------------
template <class A, bool LARGE>
__device__ __forceinline__ void cols_fwd_body(u64 *lds, u64 *p, const u64 *ps, const NttTables &t, int mi, int n, int n2) {
    A ar;
    ar.init(t, mi, n);
    const int c = threadIdx.x & 15, sub = threadIdx.x >> 4;
    typename A::T v[16];
    u64 raw[16];
    if (t.large) {
#pragma unroll
        for (int k = 0; k < 16; k++) raw[k] = __builtin_nontemporal_load(ps + (unsigned)((sub + 16 * k) * n2 + c));
    } else {
#pragma unroll
        for (int k = 0; k < 16; k++) raw[k] = ps[(unsigned)((sub + 16 * k) * n2 + c)];
    }
    {
        const TableTw<A> tw(ar, 1);                 // in flight together with the data
#pragma unroll
        for (int k = 0; k < 16; k++) v[k] = ar.from_lazy(raw[k]);
        radix16_fwd_tw(v, ar, tw);
    }
#pragma unroll
    for (int k = 0; k < 16; k++) lds[pad((sub + 16 * k) * 16 + c)] = ar.to_mid(v[k]);
    const TableTw<A> tw2(ar, 16 + sub);             // in flight across the exchange
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; k++) v[k] = ar.from_mid(lds[pad((16 * sub + k) * 16 + c)]);
    radix16_fwd_tw(v, ar, tw2);
#pragma unroll
    for (int k = 0; k < 16; k++) ntt_store(LARGE, p + (unsigned)((16 * sub + k) * n2 + c), ar.to_mid(v[k]));
}
template <class A, bool LARGE>
__device__ __forceinline__ void cols_inv_body(u64 *lds, u64 *p, const NttTables &t, int mi, int n, int n2) {
    A ar;
    ar.init(t, mi, n);
    const int c = threadIdx.x & 15, sub = threadIdx.x >> 4;
    typename A::T v[16];
    u64 raw[16];
    if (t.large) {
#pragma unroll
        for (int k = 0; k < 16; k++) raw[k] = __builtin_nontemporal_load(p + (unsigned)((16 * sub + k) * n2 + c));
    } else {
#pragma unroll
        for (int k = 0; k < 16; k++) raw[k] = p[(unsigned)((16 * sub + k) * n2 + c)];
    }
    {
        const TableTw<A> tw(ar, 16 + sub);          // in flight together with the data
#pragma unroll
        for (int k = 0; k < 16; k++) v[k] = ar.from_mid(raw[k]);
        radix16_inv_tw(v, ar, tw);
    }
#pragma unroll
    for (int k = 0; k < 16; k++) lds[pad((16 * sub + k) * 16 + c)] = ar.to_mid(v[k]);
    const TableTw<A> tw2(ar, 1);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; k++) v[k] = ar.from_mid(lds[pad((sub + 16 * k) * 16 + c)]);
    radix16_inv_tw(v, ar, tw2);
#pragma unroll
    for (int k = 0; k < 16; k++) ntt_store(LARGE, p + (unsigned)((sub + 16 * k) * n2 + c), ar.to_rest_inv(v[k]));
}

// grid.x = limbs * (n2/16)
template <bool LARGE>
__global__ __launch_bounds__(NTT_THREADS) void ntt_cols_fwd(u64 *__restrict__ data, const u64 *__restrict__ src,
                                                           const int *__restrict__ src_rows,
                                                           const int *__restrict__ rows,
                                                           const int *__restrict__ mod_idx, NttTables t, int n,
                                                           int n2) {
    __shared__ u64 lds[LDS_WORDS];
    const int tiles = n2 >> 4;
    const int limb = blockIdx.x / tiles, c0 = (blockIdx.x % tiles) << 4;
    const int mi = mod_idx[limb];
    u64 *p = data + (size_t)(rows ? rows[limb] : limb) * n + c0;
    const u64 *ps = src ? src + (size_t)(src_rows ? src_rows[limb] : limb) * n + c0 : p;
    if (t.fpq[mi].q != 0.0)
        cols_fwd_body<FpArith, LARGE>(lds, p, ps, t, mi, n, n2);
    else
        cols_fwd_body<IntArith, LARGE>(lds, p, ps, t, mi, n, n2);
}
template <bool LARGE>
__global__ __launch_bounds__(NTT_THREADS) void ntt_cols_inv(u64 *__restrict__ data, const int *__restrict__ rows,
                                                           const int *__restrict__ mod_idx, NttTables t, int n,
                                                           int n2) {
    __shared__ u64 lds[LDS_WORDS];
    const int tiles = n2 >> 4;
    const int limb = blockIdx.x / tiles, c0 = (blockIdx.x % tiles) << 4;
    const int mi = mod_idx[limb];
    u64 *p = data + (size_t)(rows ? rows[limb] : limb) * n + c0;
    if (t.fpq[mi].q != 0.0)
        cols_inv_body<FpArith, LARGE>(lds, p, t, mi, n, n2);
    else
        cols_inv_body<IntArith, LARGE>(lds, p, t, mi, n, n2);
}

// The exchange between the two radix-16 groups of a row pass stays among the sixteen lanes that share a block of 256 words,
// i.e. inside a wave: LDS operations of a wave are in order, so no barrier is needed (only the compiler has to keep them
// in order).  Cross-lane (DPP) moves in place of the trip cost 192 vector ALU instructions per lane in passes that are
// bound by that unit (up to 86 % busy).  With the LDS trip instead, four stages between renormalisations and the tails in
// FP64: 1112 limbs 248 -> 216 us, 368 limbs with the ModDown tail 157 -> 136 us.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// The fused ModDown / rescale tail of a forward transform: the canonical words of a chunk of CH sit in LDS.
// at(e): where word e of the chunk sits.  DROP: the rescale may be part of it (FinishBatch::ainv); at n = 4096 only the folded
// conversions end so, and the others keep their registers (eight sources: 20.2 us instead of 20.9).
template <int LANES, int CH = 4096, bool DROP = true, class AT, class A>
__device__ __forceinline__ void finish_tail(AT at, const A &ar, const u64 *lds, const NttTables &t, int n, int chunk, int limb, const FinishBatch &fb) {
    constexpr int NW = CH / LANES;
    // this limb is NTT(conv) of item r, component c, limb l
    const int per = fb.ncomp * (fb.level + 1);
    const int r = limb / per, c = fb.comp0 + (limb % per) / (fb.level + 1), l = limb % (fb.level + 1);
    const u64 pi = fb.pinv[2 * l], pis = fb.pinv[2 * l + 1];
    const unsigned pos0 = (unsigned)chunk * CH + threadIdx.x;
    const size_t row = ((size_t)c * (fb.level + 1) + l) * n, in_row = fb.in_rows ? ((size_t)c * fb.in_rows + l) * n : row;
    const u64 *up = fb.u[r] + ((size_t)c * fb.ext + l) * n + pos0;
    const u64 *ad = (fb.addend[r] && c < fb.addend_comps) ? fb.addend[r] + in_row : nullptr;
    const u64 *ac = fb.accum[r] ? fb.accum[r] + in_row + pos0 : nullptr;
    u64 *op = fb.out[r] + row + pos0;
    const unsigned g = fb.g[r];
    const int logn = 31 - __clz(n);
    // All operands of the tail are loaded first, then combined: NW independent loads per stream are in flight at
    // once instead of one load-wait-use chain per word.
    u64 uu[NW], aa[NW], cc[NW];
    if (fb.mul_pt) {
        // u = u[r] * (mul_pt through the Galois map mul_g[r]), formed here instead of being read
        const typename A::Tail tl(ar, t, l, pi, pis);
        const u64 *mp = fb.mul_pt + (size_t)l * n;
        const unsigned mg = fb.mul_g[r];
#pragma unroll
        for (int k = 0; k < NW; k++) uu[k] = up[LANES * k];
        if (mg) {
#pragma unroll
            for (int k = 0; k < NW; k++) aa[k] = mp[perm_src(pos0 + LANES * k, mg, logn)];
        } else {
#pragma unroll
            for (int k = 0; k < NW; k++) aa[k] = mp[pos0 + LANES * k];
        }
        if (ac) {
#pragma unroll
            for (int k = 0; k < NW; k++) cc[k] = TAIL_LD(ac + LANES * k);
        }
#pragma unroll
        for (int k = 0; k < NW; k++) {
            const u64 x = tl.masked(ar, uu[k], aa[k], lds[at(threadIdx.x + LANES * k)], ac != nullptr, cc[k]);
            TAIL_ST(op + LANES * k, x);
        }
        return;
    }
    const typename A::Tail tl(ar, t, l, pi, pis);
#pragma unroll
    for (int k = 0; k < NW; k++) uu[k] = up[LANES * k];
    if (ad && g) {
#pragma unroll
        for (int k = 0; k < NW; k++) aa[k] = ad[perm_src(pos0 + LANES * k, g, logn)];
    } else if (ad) {
#pragma unroll
        for (int k = 0; k < NW; k++) aa[k] = ad[pos0 + LANES * k];
    }
    if (ac) {
#pragma unroll
        for (int k = 0; k < NW; k++) cc[k] = ac[LANES * k];
    }
    if (DROP && fb.ainv && (ad || ac)) {
        const u64 ai = fb.ainv[2 * l], ais = fb.ainv[2 * l + 1];
#pragma unroll
        for (int k = 0; k < NW; k++)
            op[LANES * k] = tl.drop(ar, uu[k], lds[at(threadIdx.x + LANES * k)], ad ? aa[k] : 0, ac ? cc[k] : 0, ai, ais);
        return;
    }
#pragma unroll
    for (int k = 0; k < NW; k++) {
        const u64 x = tl.plain(ar, uu[k], lds[at(threadIdx.x + LANES * k)], ad != nullptr, aa[k], ac != nullptr, cc[k]);
        op[LANES * k] = x;
    }
}

// the words of limb `limb` (positions pos(k)) that a FoldIn turns into u + P (sigma_g(add) + acc)
template <int NW, class P>
__device__ __forceinline__ void fold_in(const FoldIn &fi, int limb, int n, int logn, u64 (&w)[NW], P pos) {
    if (!fi.per || limb % fi.per) return;
    const int c = limb / fi.per & 1, z = limb / (2 * fi.per);
    const size_t row = ((size_t)c * fi.rows + fi.rows - 1) * n;
    if (fi.add && c < fi.add_comps) {
        const u64 *a = fi.add + z * fi.add_stride + row;
#pragma unroll
        for (int k = 0; k < NW; k++) w[k] = addmod(w[k], redc((u128)a[fi.g ? perm_src(pos(k), fi.g, logn) : pos(k)] * fi.pm, fi.q, fi.qinv), fi.q);
    }
    if (fi.acc) {
        const u64 *a = fi.acc + z * fi.acc_stride + row;
#pragma unroll
        for (int k = 0; k < NW; k++) w[k] = addmod(w[k], redc((u128)a[pos(k)] * fi.pm, fi.q, fi.qinv), fi.q);
    }
}

// ---- row passes on contiguous blocks of 256 words (n = 65536): a workgroup owns 16 blocks ---------------
template <class A, bool TAIL, bool LARGE>
__device__ __forceinline__ void rows256_fwd_body(u64 *lds, u64 *p, const NttTables &t, int mi, int n, int chunk,
                                                 int limb, const FinishBatch &fb) {
    A ar;
    ar.init(t, mi, n);
    const int sub = threadIdx.x & 15, blk = threadIdx.x >> 4;
    const u64 B = (u64)chunk * 16 + blk;
    typename A::T v[16];
    u64 raw[16];
    if (t.large) {
#pragma unroll
        for (int k = 0; k < 16; k++) raw[k] = __builtin_nontemporal_load(p + blk * 256 + sub + 16 * k);
    } else {
#pragma unroll
        for (int k = 0; k < 16; k++) raw[k] = p[blk * 256 + sub + 16 * k];
    }
    {
        const TableTw<A> tw(ar, 256 + B);           // in flight together with the data
#pragma unroll
        for (int k = 0; k < 16; k++) v[k] = ar.from_mid(raw[k]);
        radix16_fwd_tw(v, ar, tw);
    }
#pragma unroll
    for (int k = 0; k < 16; k++) lds[pad(blk * 256 + sub + 16 * k)] = ar.to_mid(v[k]);
    wave_sync();
#pragma unroll
    for (int k = 0; k < 16; k++) v[k] = ar.from_mid(lds[pad(blk * 256 + 16 * sub + k)]);
    radix16_fwd_last(v, ar, 4096 + B * 16 + sub);
    // Each lane now owns 16 contiguous words.  A trip through LDS hands every lane the words tid, tid + 256, ... of the tile
    // instead, so that all global traffic below is coalesced.  A tail takes the values as they are.
#pragma unroll
    for (int k = 0; k < 16; k++) lds[pad(blk * 256 + 16 * sub + k)] = TAIL ? ar.to_tail(v[k]) : ar.to_rest_fwd(v[k]);
    __syncthreads();
    if (!TAIL) {
#pragma unroll
        for (int k = 0; k < 16; k++) ntt_store(LARGE, p + threadIdx.x + 256 * k, lds[pad(threadIdx.x + 256 * k)]);
        return;
    }
    finish_tail<NTT_THREADS>(pad, ar, lds, t, n, chunk, limb, fb);
}
template <class A, bool LARGE>
__device__ __forceinline__ void rows256_inv_body(u64 *lds, u64 *p, const u64 *ps, const u64 *psrow, unsigned g,
                                                 const NttTables &t, int mi, int n, int chunk, int limb, const FoldIn &fi) {
    A ar;
    ar.init(t, mi, n);
    const int sub = threadIdx.x & 15, blk = threadIdx.x >> 4;
    const u64 B = (u64)chunk * 16 + blk;
    typename A::T v[16];
    // coalesced load (through the Galois permutation if g != 0: a run of 64 positions maps onto one
    // aligned run of 64), then every lane picks its 16 contiguous words from LDS
    {
        const int logn = 31 - __clz(n);
        const unsigned pos0 = (unsigned)chunk * 4096 + threadIdx.x;
        u64 w[16];                        // sixteen independent loads in flight, then the writes to LDS
        if (g) {
#pragma unroll
            for (int k = 0; k < 16; k++) w[k] = psrow[perm_src(pos0 + 256 * k, g, logn)];
        } else if (t.large) {
#pragma unroll
            for (int k = 0; k < 16; k++) w[k] = __builtin_nontemporal_load(ps + threadIdx.x + 256 * k);
        } else {
#pragma unroll
            for (int k = 0; k < 16; k++) w[k] = ps[threadIdx.x + 256 * k];
        }
        if (!LARGE) fold_in(fi, limb, n, logn, w, [&](int k) { return pos0 + 256 * k; });
#pragma unroll
        for (int k = 0; k < 16; k++) lds[pad(threadIdx.x + 256 * k)] = w[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; k++) v[k] = ar.from_rest(lds[pad(blk * 256 + 16 * sub + k)]);
    }
    radix16_inv_last(v, ar, 4096 + B * 16 + sub);
    const TableTw<A> tw2(ar, 256 + B);
#pragma unroll
    for (int k = 0; k < 16; k++) lds[pad(blk * 256 + 16 * sub + k)] = ar.to_mid(v[k]);       // the words it read
    wave_sync();
#pragma unroll
    for (int k = 0; k < 16; k++) v[k] = ar.from_mid(lds[pad(blk * 256 + sub + 16 * k)]);
    radix16_inv_tw(v, ar, tw2);
#pragma unroll
    for (int k = 0; k < 16; k++) ntt_store(LARGE, p + blk * 256 + sub + 16 * k, ar.to_mid(v[k]));
}
// grid.x = limbs * n/4096; TAIL: the fused ModDown / rescale tail (a kernel of its own, so that the registers its
// operands take do not lower the occupancy of the plain transform)
template <bool TAIL, bool LARGE>
__global__ __launch_bounds__(NTT_THREADS) void ntt_rows256_fwd(u64 *__restrict__ data, const int *__restrict__ rows,
                                                              const int *__restrict__ mod_idx, NttTables t, int n,
                                                              FinishBatch fb) {
    __shared__ u64 lds[LDS_WORDS];
    const int per = n >> 12;
    const int limb = blockIdx.x / per, chunk = blockIdx.x % per;
    const int mi = mod_idx[limb];
    u64 *p = data + (size_t)(rows ? rows[limb] : limb) * n + (size_t)chunk * 4096;
    if (t.fpq[mi].q != 0.0)
        rows256_fwd_body<FpArith, TAIL, LARGE>(lds, p, t, mi, n, chunk, limb, fb);
    else
        rows256_fwd_body<IntArith, TAIL, LARGE>(lds, p, t, mi, n, chunk, limb, fb);
}
template <bool LARGE>
__global__ __launch_bounds__(NTT_THREADS) void ntt_rows256_inv(u64 *__restrict__ data, const u64 *__restrict__ src,
                                                              const int *__restrict__ src_rows,
                                                              const int *__restrict__ rows,
                                                              const int *__restrict__ mod_idx, NttTables t, int n,
                                                              unsigned g, FoldIn fi) {
    __shared__ u64 lds[LDS_WORDS];
    const int per = n >> 12;
    const int limb = blockIdx.x / per, chunk = blockIdx.x % per;
    const int mi = mod_idx[limb];
    u64 *p = data + (size_t)(rows ? rows[limb] : limb) * n + (size_t)chunk * 4096;
    const u64 *psrow = src ? src + (size_t)(src_rows ? src_rows[limb] : limb) * n : p - (size_t)chunk * 4096;
    const u64 *ps = psrow + (size_t)chunk * 4096;
    if (t.fpq[mi].q != 0.0)
        rows256_inv_body<FpArith, LARGE>(lds, p, ps, psrow, g, t, mi, n, chunk, limb, fi);
    else
        rows256_inv_body<IntArith, LARGE>(lds, p, ps, psrow, g, t, mi, n, chunk, limb, fi);
}

// ---- passes of a few limbs (n = 65536): four words a lane --------------------------------------------------------------
// With few limbs a pass takes as long as one lane's chain of loads, butterflies and exchanges: with sixteen words a lane that is
// 64 butterflies one after the other in a wave alone on its SIMD.  Here 512 lanes own 2048 words as radix 4 x 4 x 4 x 4: a
// quarter of the chain, two waves on every SIMD, twice the workgroups, for two exchanges more.  Sixteen words -> four, in us:
// 8 limbs under 60-bit primes, inverse rows 8.6 -> 6.1, columns 9.7 -> 8.4; 4 limbs below 2^50, inverse 6.4 -> 4.2 and
// 6.4 -> 5.6, forward rows 8.9 -> 5.6; 8 limbs with the ModDown tail 10.5 -> 7.4; columns of 6 limbs forward 6.7 -> 5.4.
// A rotary embedding at level 3 (three key switches): 168 -> 138 us.
// The limits: SMALL_COLS, because 64-byte segments cost columns more than the chain once there is work for every compute unit
// (14 limbs inverse 6.9 -> 11.1; sixteen columns and 1024 lanes: 9.3, and slower below); SMALL_PLAIN for forward rows
// (13 limbs 9.7 -> 8.0, 28 limbs 13.5 -> 14.0, 58 limbs 16.5 -> 18.4); SMALL_ROWS for inverse rows and forward rows with a tail
// (35 limbs inverse 14.7 -> 11.3; 64 limbs 20.0 -> 18.9 and 30.3 -> 26.5; 80 limbs with a tail the same).  All tails were
// ModDowns; full batches of an append's masked products (64 limbs a level) are past the limit and were not timed in this form.
#define SMALL_COLS 8
#define SMALL_PLAIN 16
#define SMALL_ROWS 64
#define SMALL_CW 8                // columns of a workgroup
#define SMALL_THREADS 512
#define SMALL_CHUNK 2048
// A column (or a row) of 256 words is shared by 64 lanes.  v[k] = word 64 k + sub on one side, 4 sub + k on the other;
// at(base, step, k): LDS place of word base + step k; R: 1 for the columns (stages 0..7), 256 + row for the rows (stages 8..15).
template <class A>
struct SmallTw {
    const Tw<A, 2> t0, t1, t2, t3;
    __device__ __forceinline__ SmallTw(const A &ar, unsigned R, int sub) : t0(ar, R), t1(ar, 4 * R + (sub >> 4)), t2(ar, 16 * R + (sub >> 2)), t3(ar, 64 * R + sub) {}
};
template <class A, class AT, class S>
__device__ __forceinline__ void small_fwd(u64 *lds, typename A::T (&v)[4], const A &ar, const SmallTw<A> &tw, int sub, AT at, S sync) {
    const int hi1 = sub >> 4, lo1 = sub & 15, hi2 = sub >> 2, lo2 = sub & 3;
    const Tw<A, 2> &t1 = tw.t1, &t2 = tw.t2, &t3 = tw.t3;
    radix_fwd<2, 0>(v, ar, tw.t0);
#pragma unroll
    for (int k = 0; k < 4; k++) lds[at(sub, 64, k)] = ar.to_mid(v[k]);
    sync();
#pragma unroll
    for (int k = 0; k < 4; k++) v[k] = ar.from_mid(lds[at(64 * hi1 + lo1, 16, k)]);
    radix_fwd<2, 2>(v, ar, t1);
#pragma unroll
    for (int k = 0; k < 4; k++) lds[at(64 * hi1 + lo1, 16, k)] = ar.to_mid(v[k]);
    sync();
#pragma unroll
    for (int k = 0; k < 4; k++) v[k] = ar.from_mid(lds[at(16 * hi2 + lo2, 4, k)]);
    radix_fwd<2, 4>(v, ar, t2);
#pragma unroll
    for (int k = 0; k < 4; k++) lds[at(16 * hi2 + lo2, 4, k)] = ar.to_mid(v[k]);
    sync();
#pragma unroll
    for (int k = 0; k < 4; k++) v[k] = ar.from_mid(lds[at(4 * sub, 1, k)]);
    radix_fwd<2, 6>(v, ar, t3);
}
template <class A, class AT, class S>
__device__ __forceinline__ void small_inv(u64 *lds, typename A::T (&v)[4], const A &ar, unsigned R, int sub, AT at, S sync) {
    const int hi1 = sub >> 4, lo1 = sub & 15, hi2 = sub >> 2, lo2 = sub & 3;
    const Tw<A, 2> t0(ar, R), t1(ar, 4 * R + hi1), t2(ar, 16 * R + hi2);
    radix_inv<2, 6>(v, ar, Tw<A, 2>(ar, 64 * R + sub));
#pragma unroll
    for (int k = 0; k < 4; k++) lds[at(4 * sub, 1, k)] = ar.to_mid(v[k]);
    sync();
#pragma unroll
    for (int k = 0; k < 4; k++) v[k] = ar.from_mid(lds[at(16 * hi2 + lo2, 4, k)]);
    radix_inv<2, 4>(v, ar, t2);
#pragma unroll
    for (int k = 0; k < 4; k++) lds[at(16 * hi2 + lo2, 4, k)] = ar.to_mid(v[k]);
    sync();
#pragma unroll
    for (int k = 0; k < 4; k++) v[k] = ar.from_mid(lds[at(64 * hi1 + lo1, 16, k)]);
    radix_inv<2, 2>(v, ar, t1);
#pragma unroll
    for (int k = 0; k < 4; k++) lds[at(64 * hi1 + lo1, 16, k)] = ar.to_mid(v[k]);
    sync();
#pragma unroll
    for (int k = 0; k < 4; k++) v[k] = ar.from_mid(lds[at(sub, 64, k)]);
    radix_inv<2, 0>(v, ar, t0);
}
// SMALL_CW columns of 256 words; the rows that a half-wave touches (neighbours, or four apart) cover all banks
struct SmallCol {
    int c;
    __device__ __forceinline__ int operator()(int base, int step, int k) const {
        const int e = base + step * k;
        return SMALL_CW * (e ^ ((e >> 2) & (32 / SMALL_CW - 1))) + c;
    }
};
struct SmallRow {
    int row;                      // first word of the row, a multiple of 16; no step carries from below a multiple of 16 past it
    __device__ __forceinline__ int operator()(int base, int step, int k) const { return pad(row + base) + pad(step * k); }
};
struct GroupSync {
    __device__ __forceinline__ void operator()() const { __syncthreads(); }
};
struct WaveSync {
    __device__ __forceinline__ void operator()() const { wave_sync(); }
};
template <class A>
__device__ __forceinline__ void small_cols_fwd_body(u64 *lds, u64 *p, const u64 *ps, const NttTables &t, int mi, int n) {
    A ar;
    ar.init(t, mi, n);
    const int n2 = n >> 8, c = threadIdx.x % SMALL_CW, sub = threadIdx.x / SMALL_CW;
    u64 raw[4];
    typename A::T v[4];
#pragma unroll
    for (int k = 0; k < 4; k++) raw[k] = ps[(64 * k + sub) * n2 + c];
#pragma unroll
    for (int k = 0; k < 4; k++) v[k] = ar.from_lazy(raw[k]);
    small_fwd(lds, v, ar, SmallTw<A>(ar, 1, sub), sub, SmallCol{c}, GroupSync());
#pragma unroll
    for (int k = 0; k < 4; k++) ntt_store(0, p + (4 * sub + k) * n2 + c, ar.to_mid(v[k]));
}
template <class A>
__device__ __forceinline__ void small_cols_inv_body(u64 *lds, u64 *p, const NttTables &t, int mi, int n) {
    A ar;
    ar.init(t, mi, n);
    const int n2 = n >> 8, c = threadIdx.x % SMALL_CW, sub = threadIdx.x / SMALL_CW;
    typename A::T v[4];
#pragma unroll
    for (int k = 0; k < 4; k++) v[k] = ar.from_mid(p[(4 * sub + k) * n2 + c]);
    small_inv(lds, v, ar, 1, sub, SmallCol{c}, GroupSync());
#pragma unroll
    for (int k = 0; k < 4; k++) ntt_store(0, p + (64 * k + sub) * n2 + c, ar.to_rest_inv(v[k]));
}
// eight rows, a wave each: the exchanges stay inside it
template <class A, bool TAIL>
__device__ __forceinline__ void small_rows_fwd_body(u64 *lds, u64 *p, const NttTables &t, int mi, int n, int chunk, int limb,
                                                    const FinishBatch &fb) {
    A ar;
    ar.init(t, mi, n);
    const int sub = threadIdx.x & 63, row = threadIdx.x >> 6;
    p += row * 256;
    typename A::T v[4];
#pragma unroll
    for (int k = 0; k < 4; k++) v[k] = ar.from_mid(p[64 * k + sub]);
    small_fwd(lds, v, ar, SmallTw<A>(ar, 256 + 8 * chunk + row, sub), sub, SmallRow{row * 256}, WaveSync());
#pragma unroll
    for (int k = 0; k < 4; k++) lds[pad(row * 256 + 4 * sub + k)] = TAIL ? ar.to_tail(v[k]) : ar.to_rest_fwd(v[k]);
    if (!TAIL) {
        wave_sync();
#pragma unroll
        for (int k = 0; k < 4; k++) ntt_store(0, p + 64 * k + sub, lds[pad(row * 256 + 64 * k + sub)]);
        return;
    }
    __syncthreads();
    finish_tail<SMALL_THREADS, SMALL_CHUNK>(pad, ar, lds, t, n, chunk, limb, fb);
}
template <class A>
__device__ __forceinline__ void small_rows_inv_body(u64 *lds, u64 *p, const u64 *psrow, unsigned g, const NttTables &t, int mi, int n,
                                                    int chunk, int limb, const FoldIn &fi) {
    A ar;
    ar.init(t, mi, n);
    const int sub = threadIdx.x & 63, row = threadIdx.x >> 6, logn = 31 - __clz(n);
    const unsigned pos0 = (unsigned)chunk * SMALL_CHUNK + row * 256 + 4 * sub;
    u64 raw[4];
    typename A::T v[4];
#pragma unroll
    for (int k = 0; k < 4; k++) raw[k] = psrow[g ? perm_src(pos0 + k, g, logn) : pos0 + k];
    fold_in(fi, limb, n, logn, raw, [&](int k) { return pos0 + k; });
#pragma unroll
    for (int k = 0; k < 4; k++) v[k] = ar.from_rest(raw[k]);
    small_inv(lds, v, ar, 256 + 8 * chunk + row, sub, SmallRow{row * 256}, WaveSync());
#pragma unroll
    for (int k = 0; k < 4; k++) ntt_store(0, p + row * 256 + 64 * k + sub, ar.to_mid(v[k]));
}
// grid.x = limbs * n / 2048
__global__ __launch_bounds__(64 * SMALL_CW) void small_cols_fwd(u64 *__restrict__ data, const u64 *__restrict__ src,
                                                               const int *__restrict__ src_rows, const int *__restrict__ rows,
                                                               const int *__restrict__ mod_idx, NttTables t, int n) {
    __shared__ u64 lds[256 * SMALL_CW];
    const int per = n / (256 * SMALL_CW), limb = blockIdx.x / per, c0 = (blockIdx.x % per) * SMALL_CW, mi = mod_idx[limb];
    u64 *p = data + (size_t)(rows ? rows[limb] : limb) * n + c0;
    const u64 *ps = src ? src + (size_t)(src_rows ? src_rows[limb] : limb) * n + c0 : p;
    if (t.fpq[mi].q != 0.0) small_cols_fwd_body<FpArith>(lds, p, ps, t, mi, n);
    else small_cols_fwd_body<IntArith>(lds, p, ps, t, mi, n);
}
__global__ __launch_bounds__(64 * SMALL_CW) void small_cols_inv(u64 *__restrict__ data, const int *__restrict__ rows,
                                                               const int *__restrict__ mod_idx, NttTables t, int n) {
    __shared__ u64 lds[256 * SMALL_CW];
    const int per = n / (256 * SMALL_CW), limb = blockIdx.x / per, c0 = (blockIdx.x % per) * SMALL_CW, mi = mod_idx[limb];
    u64 *p = data + (size_t)(rows ? rows[limb] : limb) * n + c0;
    if (t.fpq[mi].q != 0.0) small_cols_inv_body<FpArith>(lds, p, t, mi, n);
    else small_cols_inv_body<IntArith>(lds, p, t, mi, n);
}
template <bool TAIL>
__global__ __launch_bounds__(SMALL_THREADS) void small_rows_fwd(u64 *__restrict__ data, const int *__restrict__ rows,
                                                               const int *__restrict__ mod_idx, NttTables t, int n, FinishBatch fb) {
    __shared__ u64 lds[SMALL_CHUNK + SMALL_CHUNK / 16];
    const int per = n / SMALL_CHUNK, limb = blockIdx.x / per, chunk = blockIdx.x % per, mi = mod_idx[limb];
    u64 *p = data + (size_t)(rows ? rows[limb] : limb) * n + (size_t)chunk * SMALL_CHUNK;
    if (t.fpq[mi].q != 0.0) small_rows_fwd_body<FpArith, TAIL>(lds, p, t, mi, n, chunk, limb, fb);
    else small_rows_fwd_body<IntArith, TAIL>(lds, p, t, mi, n, chunk, limb, fb);
}
__global__ __launch_bounds__(SMALL_THREADS) void small_rows_inv(u64 *__restrict__ data, const u64 *__restrict__ src,
                                                               const int *__restrict__ src_rows, const int *__restrict__ rows,
                                                               const int *__restrict__ mod_idx, NttTables t, int n, unsigned g, FoldIn fi) {
    __shared__ u64 lds[SMALL_CHUNK + SMALL_CHUNK / 16];
    const int per = n / SMALL_CHUNK, limb = blockIdx.x / per, chunk = blockIdx.x % per, mi = mod_idx[limb];
    u64 *p = data + (size_t)(rows ? rows[limb] : limb) * n + (size_t)chunk * SMALL_CHUNK;
    const u64 *psrow = src ? src + (size_t)(src_rows ? src_rows[limb] : limb) * n : p - (size_t)chunk * SMALL_CHUNK;
    if (t.fpq[mi].q != 0.0) small_rows_inv_body<FpArith>(lds, p, psrow, g, t, mi, n, chunk, limb, fi);
    else small_rows_inv_body<IntArith>(lds, p, psrow, g, t, mi, n, chunk, limb, fi);
}

// an empty statement that the compiler must take as a new value of x: values derived from x are not loop-invariant
#define OPAQUE(x) asm volatile("" : "+v"(x))

// ---- row pass of the digits and inner product with the keys in one launch (n = 65536) -----------------------------------------
// A wave owns one row of 256 words of one limb of one output: for every item and digit it does the digit's row pass (four words a
// lane, exchanges inside the wave, no barrier), which leaves four consecutive words in every lane -- the positions whose key words
// it then reads -- and multiplies.  With a Galois element the wave transforms the row that the map takes its own row from (aligned
// blocks go to aligned blocks) and exchanges once more.  The digits' row pass as a launch of its own wrote and re-read every digit.
// The rows from inv_from on go straight into the row pass of the inverse transform, whose order of words is the one they are in.
// Bound by the latency that two waves a SIMD leave open: counters of the seven giant steps and of the shared rotations of q K^T show
// the vector ALU 0.56 to 0.61 busy, 0.35 to 0.40 of the waves' time waiting, and two conflict cycles to an LDS cycle.  239 vector
// registers (244 in the shared-key form; sums, twiddles, and the next digit requested ahead, which is worth 1 %), 95 (71) scalar ones
// spilled into lanes: the two arithmetics in one kernel.  Three waves spill 26 vector registers and lose 3 to
// 10 %, four lose 20 %.  Row passes and inner products in launches of
// their own -> here: the seven giant steps at level 22 195 + 236 -> 388 us; two launches a key switch fewer: ciphertext product at
// level 13 151.6 -> 145.6 us, rotary embedding at level 3 82.9 -> 76.9, query times K at level 12 16730 -> 16020, scores times V at
// level 22 4082 -> 3852, 4096 x 4096 product at level 23 4738 -> 4532.  Eight relinearisations with one key at level 22, inverse row
// pass included: 218 + 205 + 25 in launches of their own, 459 with the draws of every output formed anew, 382 with them kept in LDS.
// At the lower levels the launch by itself is no shorter than the three (at level 9 132, 159 and 145, at level 3 56, 78 and 64), the
// calls are: with their relinearisations in three launches and joined, scores times V at levels 13, 9, 6 and 3 2340 -> 2306, 1689 -> 1677,
// 1186 -> 1179 and 737 -> 736 us, query times K over 32 key ciphertexts at levels 9, 5 and 3 7142 -> 7075, 4313 -> 4235 and 2402 -> 2409,
// with no shared rotations at level 3 3566 -> 3589.
#define RIP_WAVES 4
#define RIP_ROW (256 + 16)
typedef u64 u64x2_t __attribute__((ext_vector_type(2)));
// Sums of products d w and d v, w in multiplier form, v a raw draw.  LAZY: they run over all items of an output (each term is below
// 2^57 and an accumulator holds 128); the integer limbs' are reduced item by item (eight terms below q 2^64 fit 128 bits).
struct RipFp {
    static constexpr bool LAZY = true;
    Acc50 b, a;
    __device__ __forceinline__ void mac(u64 d, u64 w, u64 v) {
        const unsigned d0 = (unsigned)d & LOW25, d1 = (unsigned)(d >> 25);
        b.mac(d0, d1, w), a.mac(d0, d1, v);
    }
    __device__ __forceinline__ void mac_b(u64 d, u64 w) { b.mac((unsigned)d & LOW25, (unsigned)(d >> 25), w); }
    __device__ __forceinline__ u64 sum_b(const ModC &m) const { return redc(b.total(), m.q, m.qinv); }
    __device__ __forceinline__ u64 sum_a(const ModC &m) const { return redc_raw(a.total(), m); }
};
struct RipInt {
    static constexpr bool LAZY = false;
    u128 b = 0, a = 0;
    __device__ __forceinline__ void mac(u64 d, u64 w, u64 v) { b += (u128)d * w, a += (u128)d * v; }
    __device__ __forceinline__ void mac_b(u64 d, u64 w) { b += (u128)d * w; }
    __device__ __forceinline__ u64 sum_b(const ModC &m) const { return redc(b, m.q, m.qinv); }
    __device__ __forceinline__ u64 sum_a(const ModC &m) const { return redc_raw(a, m); }
};
struct RipArgs {
    int beta, ext, level, alpha, L, nmod, n, logn, kdig, inv_from;
    const u64 *ubound, *pmont;
};
// words k of the wave's row in out, or, from inv_from on, the row pass of the inverse transform of them
template <class A>
__device__ __forceinline__ void rip_out(u64 *lds, u64 *out, const u64 (&x)[4], const RipArgs &p, const NttTables &ti, int r, int mi, unsigned R, int sub) {
    if (!p.inv_from || r < p.inv_from) {
#pragma unroll
        for (int k = 0; k < 4; k += 2) {
            const u64x2_t w = {x[k], x[k + 1]};
            *reinterpret_cast<u64x2_t *>(word_at(out + 256 * R, 4 * sub + k)) = w;
        }
        return;
    }
    A ai;
    ai.init(ti, mi, p.n);
    typename A::T v[4];
#pragma unroll
    for (int k = 0; k < 4; k++) v[k] = ai.from_rest(x[k]);
    wave_sync();
    small_inv(lds, v, ai, 256 + R, sub, SmallRow{0}, WaveSync());
#pragma unroll
    for (int k = 0; k < 4; k++) ntt_store(0, word_at(out + 256 * R, sub + 64 * k), ai.to_mid(v[k]));
}
// SHARED: one key for all outputs (one item each, no Galois element): the wave runs over outputs z0 .. z1-1, draws the uniform half
// of its key words once into LDS and keeps the twiddles.
template <class A, class S, bool SHARED>
__device__ __forceinline__ void rip_body(u64 *lds, const IpBatch &b, const RipArgs &p, const FoldIn &fi, const NttTables &t, const NttTables &ti,
                                         int r, int mi, unsigned R, int z0, int z1) {
    const ModC m = t.modc[mi];
    const int n = p.n, sub = threadIdx.x & 63, special = p.ext - p.level - 1, out_rows = b.apart ? p.ext + (b.nsum - 1) * special : p.ext;
    const unsigned pos = 256 * R + 4 * sub;
    const u64 bound = p.ubound[mi];
    const SmallRow at{0};
    const bool apart = b.apart && r > p.level;
    // addresses: uniform bases and 32-bit offsets; the draws' counters: a lane's part and a uniform one
    const u64 gv = (u64)(4 * sub) * GOLD;
    A ar;
    ar.init(t, mi, n);
    S acc[4];
    u64 r0[4], r1[4];                                     // what the sums leave, integer limbs: item by item
    // The words of digit j of item s, half-transformed (or, of the digit that holds limb r itself, as they are), and of its key:
    // requested one digit ahead.
    const int jo = r <= p.level ? r / p.alpha : -1;
    u64 raw[4];
    u64x2_t w01, w23;
    auto request = [&](int z, int s, int j) {
        const IpItem &it = b.it[z * b.nsum + s];
        const u64 *kb = it.key + ((size_t)j * p.nmod + mi) * n + 256 * R;
        if (j == jo) {
            const unsigned gg = it.g ? it.g : it.own_g;
            unsigned ps = pos;
            OPAQUE(ps);                                   // what the rarer branches derive from it is not kept over the loop
#pragma unroll
            for (int k = 0; k < 4; k++) raw[k] = *word_at(it.own + (size_t)r * n, gg ? perm_src(ps + k, gg, p.logn) : ps + k);
        } else {
            const u64 *h = it.dig + ((size_t)j * p.ext + r) * n + (it.g ? perm_src(256 * R, it.g, p.logn) & ~255u : 256 * R);
#pragma unroll
            for (int k = 0; k < 4; k++) raw[k] = __builtin_nontemporal_load(word_at(h, 64 * k + sub));
        }
        const u64x2_t *k01 = reinterpret_cast<const u64x2_t *>(word_at(kb, 4 * sub)), *k23 = reinterpret_cast<const u64x2_t *>(word_at(kb, 4 * sub + 2));
        if (SHARED) w01 = *k01, w23 = *k23;               // read again for the next output
        else w01 = __builtin_nontemporal_load(k01), w23 = __builtin_nontemporal_load(k23);
    };
    auto stream_key = [&](const IpItem &it, int j) { return it.key[(size_t)p.kdig * p.nmod * n + (size_t)j * p.nmod + mi]; };
    auto draws = [&](u64 sk, u64 (&v)[4]) {
        bool rej = false;
#pragma unroll
        for (int k = 0; k < 4; k++) v[k] = mix64(gv + (sk + ((u64)(256 * R + k) + 1) * GOLD)), rej |= v[k] >= bound;
        if (rej) {
            unsigned ps = pos;
            OPAQUE(ps);
#pragma unroll
            for (int k = 0; k < 4; k++) v[k] = evk_a_draw(sk, ((u64)(ps + k) + 1) * GOLD, ps + k, bound);
        }
    };
    u64x2_t *drawn = reinterpret_cast<u64x2_t *>(lds + RIP_ROW) + 2 * sub;           // a lane's own words
    if (SHARED) {
        for (int j = 0; j < p.beta; j++) {
            u64 v[4];
            draws(stream_key(b.it[z0], j), v);
            drawn[128 * j] = u64x2_t{v[0], v[1]}, drawn[128 * j + 1] = u64x2_t{v[2], v[3]};
        }
    }
    request(z0, 0, 0);
    for (int z = z0; z < (SHARED ? z1 : z0 + 1); z++) {
#pragma unroll
        for (int k = 0; k < 4; k++) r0[k] = r1[k] = 0;
        for (int s = 0; s < b.nsum; s++) {
            const IpItem &it = b.it[z * b.nsum + s];
            const unsigned g = it.g, src_row = g ? perm_src(256 * R, g, p.logn) >> 8 : R;
            const SmallTw<A> tw(ar, 256 + src_row, sub);
            for (int j = 0; j < p.beta; j++) {
                const u64 sk = SHARED ? 0 : stream_key(it, j);
                u64 d[4];
                typename A::T x[4];
                const u64 wk[4] = {w01.x, w01.y, w23.x, w23.y};
#pragma unroll
                for (int k = 0; k < 4; k++) d[k] = raw[k], x[k] = ar.from_mid(raw[k]);
                if (j + 1 < p.beta) request(z, s, j + 1);
                else if (s + 1 < b.nsum) request(z, s + 1, 0);
                else if (SHARED && z + 1 < z1) request(z + 1, 0, 0);
                unsigned ps = pos;
                OPAQUE(ps);
                if (j != jo) {
                    wave_sync();
                    small_fwd(lds, x, ar, tw, sub, at, WaveSync());
#pragma unroll
                    for (int k = 0; k < 4; k++) d[k] = ar.to_rest_fwd(x[k]);
                    if (g) {
                        wave_sync();
#pragma unroll
                        for (int k = 0; k < 4; k++) lds[at(4 * sub, 1, k)] = d[k];
                        wave_sync();
#pragma unroll
                        for (int k = 0; k < 4; k++) d[k] = lds[pad(perm_src(ps + k, g, p.logn) & 255)];
                    }
                }
                u64 v[4];
                if (SHARED) {
                    const u64x2_t v01 = drawn[128 * j], v23 = drawn[128 * j + 1];
                    v[0] = v01.x, v[1] = v01.y, v[2] = v23.x, v[3] = v23.y;
                } else {
                    draws(sk, v);
                }
#pragma unroll
                for (int k = 0; k < 4; k++) acc[k].mac(d[k], wk[k], v[k]);
            }
            if (it.c0 && (it.c0_ext || r <= p.level)) {
                const u64 w = it.c0_ext ? redc((u128)m.r2, m.q, m.qinv) : p.pmont[r];        // 1 or P in multiplier form
#pragma unroll
                for (int k = 0; k < 4; k++) acc[k].mac_b(*word_at(it.c0 + (size_t)r * n, g ? perm_src(pos + k, g, p.logn) : pos + k), w);
            }
            if (!S::LAZY || apart || s + 1 == b.nsum) {
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const u64 x = acc[k].sum_b(m), y = acc[k].sum_a(m);
                    r0[k] = S::LAZY ? x : addmod(r0[k], x, m.q), r1[k] = S::LAZY ? y : addmod(r1[k], y, m.q);
                    acc[k] = S();
                }
            }
            if (apart) {                                      // this item's special limb by itself
                u64 *out = b.out[z] + (size_t)(r + s * special) * n;
                rip_out<A>(lds, out, r0, p, ti, r, mi, R, sub);
                rip_out<A>(lds, out + (size_t)out_rows * n, r1, p, ti, r, mi, R, sub);
#pragma unroll
                for (int k = 0; k < 4; k++) r0[k] = r1[k] = 0;
            }
        }
        if (apart) continue;
        if (b.extra[z]) {
            const u64 *e = b.extra[z] + (size_t)r * n;
#pragma unroll
            for (int k = 0; k < 4; k++)
                r0[k] = addmod(r0[k], *word_at(e, pos + k), m.q), r1[k] = addmod(r1[k], *word_at(e + (size_t)out_rows * n, pos + k), m.q);
        }
        if (fi.per && r == p.level) {
#pragma unroll
            for (int c = 0; c < 2; c++) {
                const size_t row = ((size_t)c * fi.rows + fi.rows - 1) * n;
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    u64 x = 0;
                    if (fi.add && c < fi.add_comps) x = fi.add[z * fi.add_stride + row + (fi.g ? perm_src(pos + k, fi.g, p.logn) : pos + k)];
                    if (fi.acc) x = addmod(x, fi.acc[z * fi.acc_stride + row + pos + k], m.q);
                    x = redc((u128)x * fi.pm, m.q, m.qinv);
                    if (c) r1[k] = addmod(r1[k], x, m.q);
                    else r0[k] = addmod(r0[k], x, m.q);
                }
            }
        }
        u64 *out = b.out[z] + (size_t)r * n;
        rip_out<A>(lds, out, r0, p, ti, r, mi, R, sub);
        rip_out<A>(lds, out + (size_t)out_rows * n, r1, p, ti, r, mi, R, sub);
    }
}
// grid: x = 64 workgroups of four rows, y = limb (special primes first), z = output, or a run of `per` outputs with one key
template <bool SHARED>
__global__ CODE_ALIGN __launch_bounds__(64 * RIP_WAVES, 2) void k_rows_ip(IpBatch b, RipArgs p, FoldIn fi, NttTables t, NttTables ti, int per) {
    extern __shared__ u64 lds[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r = p.ext - 1 - (int)blockIdx.y;
    const int mi = r <= p.level ? r : p.L + 1 + (r - p.level - 1);
    u64 *l = lds + wave * (RIP_ROW + (SHARED ? 256 * p.beta : 0));
    const unsigned R = blockIdx.x * RIP_WAVES + wave;
    const int z0 = blockIdx.z * per, z1 = min(z0 + per, b.nz);
    if (t.fpq[mi].q != 0.0) rip_body<FpArith, RipFp, SHARED>(l, b, p, fi, t, ti, r, mi, R, z0, z1);
    else rip_body<IntArith, RipInt, SHARED>(l, b, p, fi, t, ti, r, mi, R, z0, z1);
}

// Row pass of the inverse transform of the last limbs of a cache append's masked products, formed on load: limb 2 z + c is
// src_z[c] (its last limb) times the mask through the Galois map g_z.  As a launch of its own the product wrote and re-read its
// limbs: 13.2 + 19.3 us for 32 products at level 4, here 17.5.
template <class A>
__device__ __forceinline__ void small_rows_inv_mul_body(u64 *lds, u64 *p, const u64 *src, const u64 *pt, unsigned g, const NttTables &t, int mi, int n, int chunk) {
    A ar;
    ar.init(t, mi, n);
    const ModC m = t.modc[mi];
    const int sub = threadIdx.x & 63, row = threadIdx.x >> 6, logn = 31 - __clz(n);
    const unsigned pos0 = (unsigned)chunk * SMALL_CHUNK + row * 256 + 4 * sub;
    u64 a[4], b[4];
    typename A::T v[4];
#pragma unroll
    for (int k = 0; k < 4; k++) a[k] = src[pos0 + k], b[k] = pt[g ? perm_src(pos0 + k, g, logn) : pos0 + k];
#pragma unroll
    for (int k = 0; k < 4; k++) v[k] = ar.from_rest(redc((u128)a[k] * b[k], m.q, m.qinv));
    small_inv(lds, v, ar, 256 + 8 * chunk + row, sub, SmallRow{row * 256}, WaveSync());
#pragma unroll
    for (int k = 0; k < 4; k++) ntt_store(0, p + row * 256 + 64 * k + sub, ar.to_mid(v[k]));
}
__global__ __launch_bounds__(SMALL_THREADS) void small_rows_inv_mul(u64 *__restrict__ data, MulPtBatch b, const u64 *__restrict__ pt, int mi, int limbs,
                                                                   NttTables t, int n) {
    __shared__ u64 lds[SMALL_CHUNK + SMALL_CHUNK / 16];
    const int per = n / SMALL_CHUNK, limb = blockIdx.x / per, chunk = blockIdx.x % per, z = limb >> 1, c = limb & 1;
    u64 *p = data + (size_t)limb * n + (size_t)chunk * SMALL_CHUNK;
    const u64 *src = b.src[z] + ((size_t)c * limbs + limbs - 1) * n, *m = pt + (size_t)(limbs - 1) * n;
    if (t.fpq[mi].q != 0.0) small_rows_inv_mul_body<FpArith>(lds, p, src, m, b.g[z], t, mi, n, chunk);
    else small_rows_inv_mul_body<IntArith>(lds, p, src, m, b.g[z], t, mi, n, chunk);
}

// ---- the whole transform of a limb of 4096 words (n = 4096) in one workgroup ---------------------------------
// 512 lanes with eight words each run the twelve stages as radix 8 x 8 x 8 x 8, all exchanges in LDS.  Bound by the chain of
// its stages, not by bytes (32 KiB per limb): as a column and a row pass the limb took two launches, and at 2 to 25 limbs
// a launch costs its few microseconds whatever it moves.  Eight words a lane keep two waves on every SIMD of the one
// compute unit a limb has; with 256 lanes of sixteen words each wave is alone on its SIMD and waits out every latency.
// A 64 x 64 product on the 5 + 1 ring (11 rotations): 693 us with two passes and separate conversion and tail, 562 us with
// whole limbs and the tail, 483 us with eight words a lane and the conversion in front.
#define FULL_THREADS 512
#define FULL_LDS (4096 + 512)
// one pad word per eight: lanes eight words apart, and runs of eight 64 words apart, hit distinct banks
__device__ __forceinline__ int pad8(int e) { return e + (e >> 3); }
// v[k] = word tid + 512 k
template <class A, bool TAIL, bool DROP = false>
__device__ __forceinline__ void full_fwd_body(u64 *lds, u64 *p, typename A::T (&v)[8], const A &ar, const NttTables &t, int n, int limb,
                                              const FinishBatch &fb) {
    const int tid = threadIdx.x, h2 = tid >> 6, l2 = tid & 63, h3 = tid >> 3, l3 = tid & 7;
    {
        const Tw<A, 3> tw(ar, 1);
        radix_fwd<3, 0>(v, ar, tw);
    }
#pragma unroll
    for (int k = 0; k < 8; k++) lds[pad8(k * 512 + tid)] = ar.to_mid(v[k]);
    {
        const Tw<A, 3> tw(ar, 8 + h2);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 8; k++) v[k] = ar.from_mid(lds[pad8(h2 * 512 + k * 64 + l2)]);
        radix_fwd<3, 3>(v, ar, tw);
    }
    // every lane writes back the words it read, so one barrier per exchange is enough
#pragma unroll
    for (int k = 0; k < 8; k++) lds[pad8(h2 * 512 + k * 64 + l2)] = ar.to_mid(v[k]);
    {
        const Tw<A, 3> tw(ar, 64 + h3);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 8; k++) v[k] = ar.from_mid(lds[pad8(h3 * 64 + k * 8 + l3)]);
        radix_fwd<3, 6>(v, ar, tw);
    }
#pragma unroll
    for (int k = 0; k < 8; k++) lds[pad8(h3 * 64 + k * 8 + l3)] = ar.to_mid(v[k]);
    {
        const Tw<A, 3> tw(ar, 512 + tid);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 8; k++) v[k] = ar.from_mid(lds[pad8(tid * 8 + k)]);
        radix_fwd<3, 9>(v, ar, tw);
    }
#pragma unroll
    for (int k = 0; k < 8; k++) lds[pad8(tid * 8 + k)] = TAIL ? ar.to_tail(v[k]) : ar.to_rest_fwd(v[k]);
    __syncthreads();
    if (TAIL) {
        finish_tail<FULL_THREADS, 4096, DROP>(pad8, ar, lds, t, n, 0, limb, fb);
        return;
    }
#pragma unroll
    for (int k = 0; k < 8; k++) p[tid + 512 * k] = lds[pad8(tid + 512 * k)];
}
// up to the last factor: v[k] = word tid + 512 k, whose place in lds no other lane touches any more
template <class A>
__device__ __forceinline__ void full_inv_regs(u64 *lds, typename A::T (&v)[8], const A &ar, const u64 *ps, unsigned g, int n, int limb, const FoldIn &fi) {
    const int tid = threadIdx.x, h2 = tid >> 6, l2 = tid & 63, h3 = tid >> 3, l3 = tid & 7;
    {
        const int logn = 31 - __clz(n);
        u64 w[8];
#pragma unroll
        for (int k = 0; k < 8; k++) w[k] = ps[g ? perm_src((unsigned)(tid + 512 * k), g, logn) : tid + 512 * k];
        fold_in(fi, limb, n, logn, w, [&](int k) { return (unsigned)(tid + 512 * k); });
#pragma unroll
        for (int k = 0; k < 8; k++) lds[pad8(tid + 512 * k)] = w[k];
        const Tw<A, 3> tw(ar, 512 + tid);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 8; k++) v[k] = ar.from_rest(lds[pad8(tid * 8 + k)]);
        radix_inv<3, 9>(v, ar, tw);
    }
#pragma unroll
    for (int k = 0; k < 8; k++) lds[pad8(tid * 8 + k)] = ar.to_mid(v[k]);
    {
        const Tw<A, 3> tw(ar, 64 + h3);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 8; k++) v[k] = ar.from_mid(lds[pad8(h3 * 64 + k * 8 + l3)]);
        radix_inv<3, 6>(v, ar, tw);
    }
#pragma unroll
    for (int k = 0; k < 8; k++) lds[pad8(h3 * 64 + k * 8 + l3)] = ar.to_mid(v[k]);
    {
        const Tw<A, 3> tw(ar, 8 + h2);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 8; k++) v[k] = ar.from_mid(lds[pad8(h2 * 512 + k * 64 + l2)]);
        radix_inv<3, 3>(v, ar, tw);
    }
#pragma unroll
    for (int k = 0; k < 8; k++) lds[pad8(h2 * 512 + k * 64 + l2)] = ar.to_mid(v[k]);
    {
        const Tw<A, 3> tw(ar, 1);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 8; k++) v[k] = ar.from_mid(lds[pad8(k * 512 + tid)]);
        radix_inv<3, 0>(v, ar, tw);
    }
}
template <class A>
__device__ __forceinline__ void full_inv_body(u64 *lds, u64 *p, const u64 *ps, unsigned g, const NttTables &t, int mi, int n, int limb,
                                              const FoldIn &fi) {
    A ar;
    ar.init(t, mi, n);
    typename A::T v[8];
    full_inv_regs(lds, v, ar, ps, g, n, limb, fi);
#pragma unroll
    for (int k = 0; k < 8; k++) p[k * 512 + threadIdx.x] = ar.to_rest_inv(v[k]);
}
// grid.x = limbs.  The transform may run in place: every word is read before the first is written.
template <class A, bool TAIL>
__device__ __forceinline__ void full_fwd_load(u64 *lds, u64 *p, const u64 *ps, const NttTables &t, int mi, int n, int limb,
                                              const FinishBatch &fb) {
    A ar;
    ar.init(t, mi, n);
    typename A::T v[8];
    u64 raw[8];
#pragma unroll
    for (int k = 0; k < 8; k++) raw[k] = ps[threadIdx.x + 512 * k];
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = ar.from_lazy(raw[k]);
    full_fwd_body<A, TAIL>(lds, p, v, ar, t, n, limb, fb);
}
template <bool TAIL>
__global__ __launch_bounds__(FULL_THREADS) void ntt_full_fwd(u64 *data, const u64 *src, const int *__restrict__ src_rows,
                                                            const int *__restrict__ rows, const int *__restrict__ mod_idx,
                                                            NttTables t, int n, FinishBatch fb) {
    __shared__ u64 lds[FULL_LDS];
    const int limb = blockIdx.x, mi = mod_idx[limb];
    u64 *p = data + (size_t)(rows ? rows[limb] : limb) * n;
    const u64 *ps = src ? src + (size_t)(src_rows ? src_rows[limb] : limb) * n : p;
    if (t.fpq[mi].q != 0.0)
        full_fwd_load<FpArith, TAIL>(lds, p, ps, t, mi, n, limb, fb);
    else
        full_fwd_load<IntArith, TAIL>(lds, p, ps, t, mi, n, limb, fb);
}
__global__ __launch_bounds__(FULL_THREADS) void ntt_full_inv(u64 *data, const u64 *src, const int *__restrict__ src_rows,
                                                            const int *__restrict__ rows, const int *__restrict__ mod_idx,
                                                            NttTables t, int n, unsigned g, FoldIn fi) {
    __shared__ u64 lds[FULL_LDS];
    const int limb = blockIdx.x, mi = mod_idx[limb];
    u64 *p = data + (size_t)(rows ? rows[limb] : limb) * n;
    const u64 *ps = src ? src + (size_t)(src_rows ? src_rows[limb] : limb) * n : p;
    if (t.fpq[mi].q != 0.0)
        full_inv_body<FpArith>(lds, p, ps, g, t, mi, n, limb, fi);
    else
        full_inv_body<IntArith>(lds, p, ps, g, t, mi, n, limb, fi);
}

// ---- fast base conversion, fused into the first pass of the forward transform of its results --------------------------
// in rows in_rows[m] (coefficient domain, residues under the source moduli) -> out rows out_rows[r]:
//   y_m = a_m * inv_hat_m mod q_m;  out_r = transform of sum_m y_m * hat_{m,r} mod q_r   (no correction term)
// Batch item z: table (z % tab_period)*tab_step, input at (z / in_group)*in_stride, output at z*out_stride (the digits of
// a raise use one table each and share the input; the two components of a ModDown share the table; a raise of several
// polynomials runs its digits over z % period and its polynomials over z / in_group).  If own_src is given the source rows
// of own_src (the evaluation-domain input, through the Galois map own_g if any) are copied to the same rows of the output.
struct ConvArgs {
    const ConvDev *tabs;
    int tab_step, tab_period, in_group;
    size_t in_stride, out_stride, own_stride;
    const u64 *own_src;
    unsigned own_g;
    int nt;                       // stores of the column pass: non-temporal (NttTables::large says how the passes of a transform store)
    int tg, groups;               // targets per workgroup, workgroups that convert per (tile, item) (n = 65536)
};
// The y_m of NV words.  Source moduli below 2^50 (the digits of a raise): exact integers in doubles; a product with a
// weight under an FP64 target modulus is then the butterflies' product (6 instructions and an addition per term, no
// carries), under a 60-bit one a split product (Acc50).  Larger sources (the special primes of a ModDown): 30 + 30 bit
// halves against 25 + 25 bits of the weight, again without carry chains.  Otherwise 128-bit sums.
// The integer sums are worked on one word after the other (sched_barrier): interleaving them costs more registers than a
// wave has to spare.
// FOLD: one more source, the folded last limb (ConvDev::fold).
template <int NS, int NV, bool FOLD>
struct ConvY {
    unsigned lo[NV][NS], hi[NV][NS], flo[NV], fhi[NV];
    __device__ __forceinline__ void set(const ConvDev &t, const u64 (&x)[NV][NS]) {
        if (t.split == CONV_SPLIT_25) {
#pragma unroll
            for (int m = 0; m < NS; m++) {
                const double q = t.src_qd[m], w = t.inv_hat_d[m], wq = t.inv_hat_dq[m];
#pragma unroll
                for (int k = 0; k < NV; k++) {
                    const double v = __longlong_as_double((long long)(x[k][m] | 0x4330000000000000ULL)) - TWO52;
                    const double h = v * w, l = __builtin_fma(v, w, -h), c = __builtin_rint(v * wq);
                    double y = __builtin_fma(-c, q, h) + l;                  // |y| < q
                    y += y < 0.0 ? q : 0.0;
                    lo[k][m] = (unsigned)__double2loint(y), hi[k][m] = (unsigned)__double2hiint(y);
                }
            }
            return;
        }
#pragma unroll
        for (int k = 0; k < NV; k++) {
#pragma unroll
            for (int m = 0; m < NS; m++) {
                const u64 y = mul_shoup(x[k][m], t.inv_hat[m], t.inv_hat_sh[m], t.src_q[m]);
                lo[k][m] = (unsigned)y, hi[k][m] = (unsigned)(y >> 32);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // x: the words of the folded limb, below q_level (itself below 2^50 where the sources are)
    __device__ __forceinline__ void fold(const ConvDev &t, const u64 (&x)[NV]) {
        u64 c[NV];
        const u64 q = t.fold.t.q;
        target<false>(t.split, t.fold.t, c);
#pragma unroll
        for (int k = 0; k < NV; k++) {
            const u64 y = mul_shoup(submod(x[k], c[k], q), t.fold.pinv, t.fold.pinv_sh, q);
            const double d = __longlong_as_double((long long)(y | 0x4330000000000000ULL)) - TWO52;
            flo[k] = t.split == CONV_SPLIT_25 ? (unsigned)__double2loint(d) : (unsigned)y;
            fhi[k] = t.split == CONV_SPLIT_25 ? (unsigned)__double2hiint(d) : (unsigned)(y >> 32);
        }
    }
    __device__ __forceinline__ double fd(int k) const { return __hiloint2double((int)fhi[k], (int)flo[k]); }
    __device__ __forceinline__ double yd(int k, int m) const { return __hiloint2double((int)hi[k][m], (int)lo[k][m]); }
    // keep what is derived from the words (64-bit pairs of their halves) from being hoisted out of a loop over the targets
    __device__ __forceinline__ void opaque() {
#pragma unroll
        for (int k = 0; k < NV; k++)
#pragma unroll
            for (int m = 0; m < NS; m++) {
                OPAQUE(lo[k][m]);
                OPAQUE(hi[k][m]);
            }
        if (FOLD) {
#pragma unroll
            for (int k = 0; k < NV; k++) {
                OPAQUE(flo[k]);
                OPAQUE(fhi[k]);
            }
        }
    }
    // targets below 2^50: |v| <= q, all that the forward stages ask (0.6 q where several sources are summed and reduced, 0.88 q
    // for one).  |y w - c q| <= 0.88 q per term (c off by three roundings of a value below 2^50), so the sum of nine terms
    // (the folded limb among them) stays below 2^53 and exact.
    __device__ __forceinline__ void target_fp(const ConvTarget &o, const FpArith &ar, double (&v)[NV]) const {
        double w[NS], wq[NS];
#pragma unroll
        for (int m = 0; m < NS; m++) w[m] = o.w[m], wq[m] = w[m] * ar.qinv;
#pragma unroll
        for (int k = 0; k < NV; k++) {
            double s = ar.mulmod(yd(k, 0), w[0], wq[0]);
#pragma unroll
            for (int m = 1; m < NS; m++) s += ar.mulmod(yd(k, m), w[m], wq[m]);
            if (FOLD) s += ar.mulmod(fd(k), o.wl, o.wl * ar.qinv);
            v[k] = NS > 1 || FOLD ? ar.norm(s) : s;
        }
    }
    __device__ __forceinline__ void target_any(int split, const ConvTarget &o, const FpArith &ar, double (&v)[NV]) const {
        if (split == CONV_SPLIT_25) {
            target_fp(o, ar, v);
        } else {
            u64 x[NV];
            target(split, o, x);
#pragma unroll
            for (int k = 0; k < NV; k++) v[k] = ar.from_rest(x[k]);
        }
    }
    template <bool WITH = FOLD>
    __device__ __forceinline__ void target(int split, const ConvTarget &o, u64 (&out)[NV]) const {
        u64 w[NS];
        const u64 q = o.q, qinv = o.qinv;
#pragma unroll
        for (int m = 0; m < NS; m++) w[m] = o.wm[m];
        if (split == CONV_SPLIT_25) {
#pragma unroll
            for (int k = 0; k < NV; k++) {
                Acc50 acc;
#pragma unroll
                for (int m = 0; m < NS; m++) {
                    const u64 y = (u64)__double_as_longlong(yd(k, m) + TWO52) & 0x000FFFFFFFFFFFFFULL;
                    acc.mac((unsigned)y & LOW25, (unsigned)(y >> 25), w[m]);
                }
                if (WITH) {
                    const u64 y = (u64)__double_as_longlong(fd(k) + TWO52) & 0x000FFFFFFFFFFFFFULL;
                    acc.mac((unsigned)y & LOW25, (unsigned)(y >> 25), o.wlm);
                }
                out[k] = redc(acc.total(), q, qinv);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else if (split == CONV_SPLIT_30) {
            // every term below 2^55
#pragma unroll
            for (int k = 0; k < NV; k++) {
                u64 t00 = 0, t01 = 0, t10 = 0, t11 = 0;
#pragma unroll
                for (int m = 0; m < NS + (WITH ? 1 : 0); m++) {
                    const u64 y = m < NS ? ((u64)hi[k][m] << 32) | lo[k][m] : ((u64)fhi[k] << 32) | flo[k], wm = m < NS ? w[m] : o.wlm;
                    const unsigned y0 = (unsigned)y & LOW30, y1 = (unsigned)(y >> 30);
                    const unsigned w0 = (unsigned)wm & LOW25, w1 = (unsigned)(wm >> 25);
                    t00 += (u64)y0 * w0, t01 += (u64)y0 * w1, t10 += (u64)y1 * w0, t11 += (u64)y1 * w1;
                }
                out[k] = redc((u128)t00 + ((u128)t01 << 25) + ((u128)t10 << 30) + ((u128)t11 << 55), q, qinv);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma unroll
            for (int k = 0; k < NV; k++) {
                u128 T = 0;
#pragma unroll
                for (int m = 0; m < NS; m++) T += (u128)(((u64)hi[k][m] << 32) | lo[k][m]) * w[m];
                if (WITH) T += (u128)(((u64)fhi[k] << 32) | flo[k]) * o.wlm;
                out[k] = redc(T, q, qinv);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
};
// The same from cut weights (ConvDev::near): the y_m are kept as their two halves, a sum over the sources is four multiply-adds a
// term into two accumulators without carries, and what q looks like takes their combination to below q + q / 16: two more
// multiply-adds and a fold.  With four sources 30 vector instructions a word; the forms above take 31 to FP64 targets and 67 to the
// 60-bit ones (half of a raise's work at the middle levels) or, from 60-bit sources, 63.  ModDown of 8 ciphertexts at level 22 (368
// limbs) 131 -> 109 us, with the rescale at level 12 (192 limbs) 89.5 -> 75, raise of 8 at level 12 (440 limbs) 130 -> 122; calls: query
// times K at level 12 15170 -> 14720 us, grouped-query attention 13340 -> 12970, ciphertext product at level 13 141 -> 138, 64 x 64 at
// n = 4096 427 -> 407.  Three workgroups a compute unit (80 registers) instead of two: the largest launches 3 % less, those of a single
// key switch 3 to 9 % more, calls 0 to 2 % more.
template <int NS, int NV, bool FOLD>
struct ConvNear {
    unsigned lo[NV][NS], hi[NV][NS], flo[NV], fhi[NV];
    __device__ __forceinline__ void set(const ConvDev &t, const u64 (&x)[NV][NS]) {
        if (t.split == CONV_SPLIT_25) {
#pragma unroll
            for (int m = 0; m < NS; m++) {
                const double q = t.src_qd[m], w = t.inv_hat_d[m], wq = t.inv_hat_dq[m];
#pragma unroll
                for (int k = 0; k < NV; k++) {
                    const double v = __longlong_as_double((long long)(x[k][m] | 0x4330000000000000ULL)) - TWO52;
                    const double h = v * w, l = __builtin_fma(v, w, -h), c = __builtin_rint(v * wq);
                    double y = __builtin_fma(-c, q, h) + l;                  // |y| < q
                    y += y < 0.0 ? q : 0.0;
                    const u64 i = (u64)__double_as_longlong(y + TWO52) & 0x000FFFFFFFFFFFFFULL;
                    lo[k][m] = (unsigned)i & LOW25, hi[k][m] = (unsigned)(i >> 25);
                }
            }
            return;
        }
#pragma unroll
        for (int k = 0; k < NV; k++) {
#pragma unroll
            for (int m = 0; m < NS; m++) {
                const u64 y = mul_shoup(x[k][m], t.inv_hat[m], t.inv_hat_sh[m], t.src_q[m]);
                lo[k][m] = (unsigned)y & LOW30, hi[k][m] = (unsigned)(y >> 30);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // one source, from what its inverse transform leaves before the last factor
    __device__ __forceinline__ void set_inv(const ConvDev &t, const FpArith &ar, const double (&v)[NV]) {
        const double w = t.inv_hat_nd, wq = w * ar.qinv;
#pragma unroll
        for (int k = 0; k < NV; k++) {
            const u64 y = ar.canon(ar.mulmod(v[k], w, wq));
            lo[k][0] = (unsigned)y & LOW25, hi[k][0] = (unsigned)(y >> 25);
        }
    }
    __device__ __forceinline__ void set_inv(const ConvDev &t, const IntArith &ar, const u64 (&v)[NV]) {
#pragma unroll
        for (int k = 0; k < NV; k++) {
            const u64 y = ar.to_rest_fwd(ar.mul(v[k], t.inv_hat_n));
            lo[k][0] = (unsigned)y & LOW30, hi[k][0] = (unsigned)(y >> 30);
        }
    }
    __device__ __forceinline__ void fold(const ConvDev &t, const u64 (&x)[NV]) {
        u64 c[NV];
        const u64 q = t.fold.t.q;
#pragma unroll
        for (int k = 0; k < NV; k++) flo[k] = fhi[k] = 0;
        opaque();
        sum<false>(t.fold.t, c);
#pragma unroll
        for (int k = 0; k < NV; k++) {
            const u64 y = mul_shoup((x[k] + 2 * q) - c[k], t.fold.pinv, t.fold.pinv_sh, q);
            const bool s25 = t.split == CONV_SPLIT_25;
            flo[k] = (unsigned)y & (s25 ? LOW25 : LOW30), fhi[k] = (unsigned)(s25 ? y >> 25 : y >> 30);
        }
    }
    // 32-bit values to the compiler: extended to 64 bits outside the loop over the targets they lose what is known of their upper halves
    __device__ __forceinline__ void opaque() {
#pragma unroll
        for (int k = 0; k < NV; k++)
#pragma unroll
            for (int m = 0; m < NS; m++) {
                OPAQUE(lo[k][m]);
                OPAQUE(hi[k][m]);
            }
        if (FOLD) {
#pragma unroll
            for (int k = 0; k < NV; k++) {
                OPAQUE(flo[k]);
                OPAQUE(fhi[k]);
            }
        }
    }
    template <bool WITH = FOLD>
    __device__ __forceinline__ void sum(const ConvTarget &o, u64 (&out)[NV]) const {
        const unsigned mlo = o.mlo, mhi = o.mhi, c = o.c, cb = o.cb, mask = (1u << cb) - 1u;
        auto fold_word = [&](u64 v) { return (u64)((unsigned)(v >> 32) >> cb) * c + (((u64)((unsigned)(v >> 32) & mask) << 32) | (unsigned)v); };
#pragma unroll
        for (int k = 0; k < NV; k++) {
            u64 l = 0, h = 0;
#pragma unroll
            for (int m = 0; m < NS; m++) {
                l += (u64)lo[k][m] * o.cut[m].w0, l += (u64)hi[k][m] * o.cut[m].v0;
                h += (u64)lo[k][m] * o.cut[m].w1, h += (u64)hi[k][m] * o.cut[m].v1;
            }
            if (WITH) {
                l += (u64)flo[k] * o.cutl.w0, l += (u64)fhi[k] * o.cutl.v0;
                h += (u64)flo[k] * o.cutl.w1, h += (u64)fhi[k] * o.cutl.v1;
            }
            out[k] = fold_word(l + (u64)(unsigned)h * mlo + (u64)(unsigned)(h >> 32) * mhi);
        }
        if (o.twice) {
#pragma unroll
            for (int k = 0; k < NV; k++) out[k] = fold_word(out[k]);
        }
    }
    __device__ __forceinline__ void target_any(int, const ConvTarget &o, const FpArith &ar, double (&v)[NV]) const {
        u64 x[NV];
        sum(o, x);
#pragma unroll
        for (int k = 0; k < NV; k++) v[k] = ar.from_rest(x[k]);
    }
    __device__ __forceinline__ void target(int, const ConvTarget &o, u64 (&out)[NV]) const { sum(o, out); }
};
// n = 65536.  A workgroup of 512 lanes owns a column tile (256 rows x 8 columns) of one item: every lane loads four words
// of each source, keeps the y_m in registers and runs over up to tg targets: conversion, then stages 0..7 as radix
// 4 x 4 x 4 x 4, the exchanges through two LDS buffers in turn (one barrier each).  The converted limbs are never stored: a
// raise used to write and re-read them between two launches.  Bound by the vector ALU and the latency of its barriers
// (two workgroups per compute unit, about 100 registers for four sources); 16 columns x 1024 lanes (one workgroup per
// compute unit) is 4 % slower on a product against the value cache, 4 columns (32-byte stores) 30 %, sixteen or eight
// words a lane run out of registers.  Measured: 1104 limbs of eight raises 188 + 242 us (conversion, column pass) -> 362 us,
// 144 limbs 28 + 37 -> 60 us, the 8 limbs of a ModDown at level 3 5.0 + 6.8 -> 8.6 us and a launch less.
// tg: 8 targets a workgroup, so that the y_m (as much work as one target) are formed once for eight; halved while the
// launch has fewer than CCF_FILL = 512 workgroups (two for each compute unit); 4 and 12 measured equal and 2 % slower.
// nt: non-temporal stores from CCF_NT converted limbs on, agent scope below (ntt_store): the passes of a plain transform gain from agent
// scope up to 255 limbs, this kernel, whose waves wait at barriers between their stores, does not.  With CCF_NT = 256, 192, 128, 64 and
// 1: 63 hoisted rotations at level 13 (224 limbs a batch) 2563, 2508, 2515, 2517 and 2509 us, at level 11 2184, 2135, 2119, 2127 and 2134;
// a rotation at level 23 (144 limbs) 182, 183, 175, 176 and 175; three hoisted ones at level 13 197, 195, 196, 194 and 204; scores times V at
// level 13 2335, 2327, 2308, 2309 and 2338.
#define CCF_NT 128
#define CCF_W 8
#define CCF_THREADS (64 * CCF_W)
#define CCF_TG 8
#define CCF_FILL 512
// LDS: row r of 8 words at row r ^ ((r >> 2) & 3): any four rows that a half-wave touches (neighbours, or four apart) then
// cover all banks
template <class A>
__device__ __forceinline__ void ccf_body(u64 *lds, int buf, int large, u64 *p, typename A::T (&v)[4], unsigned tid, const A &ar, int n2) {
    const int c = tid % CCF_W, sub = tid / CCF_W;
    u64 *A0 = lds + (buf ? 256 * CCF_W : 0) + c, *B0 = lds + (buf ? 0 : 256 * CCF_W) + c;
    {
        const Tw<A, 2> tw(ar, 1);
        radix_fwd<2, 0>(v, ar, tw);
    }
    const int sx = sub ^ ((sub >> 2) & 3);
#pragma unroll
    for (int k = 0; k < 4; k++) A0[(k * 64 + sx) * CCF_W] = ar.to_mid(v[k]);             // row 64 k + sub
    {
        const int hi = sub >> 4;
        const Tw<A, 2> tw(ar, 4 + hi);
        const int o = (hi * 64 + (sx & 15)) * CCF_W;                                     // row 64 hi + 16 k + lo
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; k++) v[k] = ar.from_mid(A0[o + k * 16 * CCF_W]);
        radix_fwd<2, 2>(v, ar, tw);
#pragma unroll
        for (int k = 0; k < 4; k++) B0[o + k * 16 * CCF_W] = ar.to_mid(v[k]);
    }
    {
        const int hi = sub >> 2, lo = sub & 3;
        const Tw<A, 2> tw(ar, 16 + hi);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; k++) v[k] = ar.from_mid(B0[(hi * 16 + k * 4 + (lo ^ k)) * CCF_W]);     // row 16 hi + 4 k + lo
        radix_fwd<2, 4>(v, ar, tw);
#pragma unroll
        for (int k = 0; k < 4; k++) A0[(hi * 16 + k * 4 + (lo ^ k)) * CCF_W] = ar.to_mid(v[k]);
    }
    {
        const Tw<A, 2> tw(ar, 64 + sub);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; k++) v[k] = ar.from_mid(A0[(sub * 4 + (k ^ (sub & 3))) * CCF_W]);     // row 4 sub + k
        radix_fwd<2, 6>(v, ar, tw);
    }
#pragma unroll
    for (int k = 0; k < 4; k++) ntt_store(large, word_at(p, (4 * sub + k) * n2 + c), ar.to_mid(v[k]));
}
template <int NS, int NV, bool FOLD, bool NEAR>
struct ConvForm {
    typedef ConvY<NS, NV, FOLD> T;
};
template <int NS, int NV, bool FOLD>
struct ConvForm<NS, NV, FOLD, true> {
    typedef ConvNear<NS, NV, FOLD> T;
};
// grid: x = column tile, y = target group (the last targets, those under the 60-bit primes, first), then the copies
template <int NS, bool FOLD, bool NEAR>
__global__ CODE_ALIGN __launch_bounds__(CCF_THREADS, FOLD && NS > 6 ? 2 : 4) void conv_cols_fwd(u64 *__restrict__ out, const u64 *__restrict__ in, ConvArgs a,
                                                               NttTables t, int n, int logn) {
    __shared__ u64 lds[2 * 256 * CCF_W];
    const ConvDev &tab = a.tabs[(blockIdx.z % a.tab_period) * a.tab_step];
    const int ns = tab.ns, nt = tab.nt, split = tab.split, n2 = n >> 8, tile = blockIdx.x;
    out += blockIdx.z * a.out_stride;
    if ((int)blockIdx.y == a.groups) {
        const u64 *src = a.own_src + (blockIdx.z / a.in_group) * a.own_stride;
        const unsigned i0 = (unsigned)tile * (256 * CCF_W) + threadIdx.x;
        for (int m = 0; m < ns; m++) {
            const size_t row = (size_t)tab.in_rows[m] * n;
            u64 w[4];
#pragma unroll
            for (int k = 0; k < 4; k++) w[k] = src[row + (a.own_g ? perm_src(i0 + CCF_THREADS * k, a.own_g, logn) : i0 + CCF_THREADS * k)];
#pragma unroll
            for (int k = 0; k < 4; k++) ntt_store(a.nt, out + row + i0 + CCF_THREADS * k, w[k]);
        }
        return;
    }
    const int r0 = (a.groups - 1 - (int)blockIdx.y) * a.tg, r1 = min(r0 + a.tg, nt);
    if (r0 >= nt) return;
    const int c = threadIdx.x % CCF_W, sub = threadIdx.x / CCF_W;
    in += (blockIdx.z / a.in_group) * a.in_stride + tile * CCF_W;
    typename ConvForm<NS, 4, FOLD, NEAR>::T y;
    {
        u64 x[4][NS], xf[4];
#pragma unroll
        for (int m = 0; m < NS; m++) {
            const u64 *row = in + (size_t)tab.in_rows[m] * n;
#pragma unroll
            for (int k = 0; k < 4; k++) x[k][m] = *word_at(row, (k * 64 + sub) * n2 + c);
        }
        if (FOLD) {
            const u64 *row = in + (size_t)tab.fold.row * n;
#pragma unroll
            for (int k = 0; k < 4; k++) xf[k] = *word_at(row, (k * 64 + sub) * n2 + c);
        }
        y.set(tab, x);
        if (FOLD) y.fold(tab, xf);
    }
    unsigned tid = threadIdx.x;
    int buf = 0;
    for (int r = r0; r < r1; r++, buf ^= 1) {
        OPAQUE(tid);                     // addresses are formed anew for every target (see ConvY)
        const ConvTarget &o = tab.t[r];
        u64 *p = out + (size_t)o.row * n + tile * CCF_W;
        y.opaque();
        if (o.qd != 0.0) {
            FpArith ar;
            ar.init(t, o.mod, n);
            double v[4];
            y.target_any(split, o, ar, v);
            ccf_body<FpArith>(lds, buf, a.nt, p, v, tid, ar, n2);
        } else {
            IntArith ar;
            ar.init(t, o.mod, n);
            u64 x[4];
            y.target(split, o, x);
            ccf_body<IntArith>(lds, buf, a.nt, p, x, tid, ar, n2);
        }
    }
}
// n = 4096: one workgroup per target limb, conversion and the whole transform.  grid: x = target, then the own rows; y = item
// INV: the workgroup does the inverse transform of its single source first (ConvBatch::inv), which leaves the source's words where the
// conversion wants them; its last factor is the conversion's first.  Every target of a digit repeats that transform, on compute units
// that have nothing else to do, and a key switch takes three launches instead of five: 6.7 + 8.8 us -> 12.1 (raise), 6.7 + 10.3 -> 14.9
// (ModDown), a gap between launches less each; 64 x 64 product at n = 4096 409 -> 357 us, 512 x 512 in the unrolled form 210 -> 190.
// All twiddles of a transform requested at its start: 13.4 and 15.6.
template <int NS, bool TAIL, bool FOLD, bool NEAR, bool INV = false>
__global__ __launch_bounds__(FULL_THREADS) void conv_full_fwd(u64 *__restrict__ out, const u64 *__restrict__ in, ConvArgs a, NttTables t, NttTables ti,
                                                             int n, int logn, FinishBatch fb) {
    __shared__ u64 lds[FULL_LDS];
    const int z = blockIdx.y, tid = threadIdx.x;
    const ConvDev &tab = a.tabs[(z % a.tab_period) * a.tab_step];
    const int ns = tab.ns, nt = tab.nt, r = blockIdx.x;
    out += z * a.out_stride;
    if (r >= nt) {
        if (!a.own_src || r >= nt + ns) return;
        const size_t row = (size_t)tab.in_rows[r - nt] * n;
        const u64 *src = a.own_src + (z / a.in_group) * a.own_stride + row;
        u64 w[8];
#pragma unroll
        for (int k = 0; k < 8; k++) w[k] = src[a.own_g ? perm_src((unsigned)(tid + 512 * k), a.own_g, logn) : tid + 512 * k];
#pragma unroll
        for (int k = 0; k < 8; k++) out[row + tid + 512 * k] = w[k];
        return;
    }
    in += (z / a.in_group) * a.in_stride;
    typename ConvForm<NS, 8, FOLD, NEAR>::T y;
    if constexpr (INV) {
        const u64 *src = in + (size_t)tab.in_rows[0] * n;
        if (tab.split == CONV_SPLIT_25) {
            FpArith ar;
            ar.init(ti, tab.src_mod, n);
            double v[8];
            full_inv_regs(lds, v, ar, src, a.own_g, n, 0, FoldIn());
            y.set_inv(tab, ar, v);
        } else {
            IntArith ar;
            ar.init(ti, tab.src_mod, n);
            u64 v[8];
            full_inv_regs(lds, v, ar, src, a.own_g, n, 0, FoldIn());
            y.set_inv(tab, ar, v);
        }
    } else {
        u64 x[8][NS], xf[8];
#pragma unroll
        for (int m = 0; m < NS; m++)
#pragma unroll
            for (int k = 0; k < 8; k++) x[k][m] = in[(size_t)tab.in_rows[m] * n + tid + 512 * k];
        if (FOLD) {
#pragma unroll
            for (int k = 0; k < 8; k++) xf[k] = in[(size_t)tab.fold.row * n + tid + 512 * k];
        }
        y.set(tab, x);
        if (FOLD) y.fold(tab, xf);
    }
    // the other form keeps its registers without: eight sources spill 60 with it, seven hoisted rotations on 16 + 8 primes 65.4 -> 67.8 us
    if (NEAR || FOLD) y.opaque();
    const ConvTarget &o = tab.t[r];
    const int limb = z * nt + r;                          // of the tail: item, component, limb
    u64 *p = out + (size_t)o.row * n;
    if (o.qd != 0.0) {
        FpArith ar;
        ar.init(t, o.mod, n);
        double v[8];
        y.target_any(tab.split, o, ar, v);
        full_fwd_body<FpArith, TAIL, FOLD>(lds, p, v, ar, t, n, limb, fb);
    } else {
        IntArith ar;
        ar.init(t, o.mod, n);
        u64 x[8];
        y.target(tab.split, o, x);
        full_fwd_body<IntArith, TAIL, FOLD>(lds, p, x, ar, t, n, limb, fb);
    }
}

static NttTables tables_of(const cm_ctx *ctx, bool inverse, int limbs) {
    NttTables t;
    t.modc = ctx->d_modc, t.fpq = ctx->d_fpq;
    t.large = limbs >= 256;
    if (!inverse) {
        t.tw = ctx->d_tw, t.twd = ctx->d_twd, t.twqd = ctx->d_twqd;
        t.ninv = nullptr, t.ninvd = t.ninvqd = nullptr;
    } else {
        t.tw = ctx->d_itw, t.twd = ctx->d_itwd, t.twqd = ctx->d_itwqd;
        t.ninv = ctx->d_ninv, t.ninvd = ctx->d_ninvd, t.ninvqd = ctx->d_ninvqd;
    }
    return t;
}
static void launch_cols_fwd(u64 *data, const u64 *src, const int *d_src_rows, const int *d_rows, const int *d_mods, const NttTables &t,
                            int n, int limbs, hipStream_t st) {
    if (limbs <= SMALL_COLS)
        hipLaunchKernelGGL(small_cols_fwd, dim3(limbs * (256 / SMALL_CW)), dim3(64 * SMALL_CW), 0, st, data, src, d_src_rows, d_rows, d_mods, t, n);
    else
        hipLaunchKernelGGL(t.large ? ntt_cols_fwd<true> : ntt_cols_fwd<false>, dim3(limbs * (n >> 12)), dim3(NTT_THREADS), 0, st, data, src, d_src_rows,
                           d_rows, d_mods, t, n, n >> 8);
}
template <bool TAIL>
static void launch_rows_fwd(u64 *data, const int *d_rows, const int *d_mods, const NttTables &t, int n, int limbs, const FinishBatch &fb,
                            hipStream_t st) {
    if (limbs <= (TAIL ? SMALL_ROWS : SMALL_PLAIN))
        hipLaunchKernelGGL(small_rows_fwd<TAIL>, dim3(limbs * (n / SMALL_CHUNK)), dim3(SMALL_THREADS), 0, st, data, d_rows, d_mods, t, n, fb);
    else
        hipLaunchKernelGGL((t.large ? ntt_rows256_fwd<TAIL, true> : ntt_rows256_fwd<TAIL, false>), dim3(limbs * (n >> 12)), dim3(NTT_THREADS), 0, st, data,
                           d_rows, d_mods, t, n, fb);
}
// data rows d_rows[i] (or i) are transformed in place; with src != nullptr the first pass reads row
// src_rows[i] (or i) of src instead, so the transform is out of place and src is left untouched.
// With g != 0 (inverse, out of place only) the source is read through the Galois permutation, i.e.
// the result is the coefficient form of the mapped polynomial.
void launch_ntt_src(cm_ctx *ctx, u64 *data, const int *d_rows, const u64 *src, const int *d_src_rows,
                    const int *d_mod_idx, int limbs, bool inverse, hipStream_t st, u64 g, const FoldIn &fi) {
    if (limbs <= 0) return;
    if (g && (!inverse || !src || src == data)) g = 0;
    Prof prof_(ctx, inverse ? CM_K_NTT_INV : CM_K_NTT_FWD, limbs, st);
    const int n = ctx->n, n2 = n >> 8;
    dim3 grid((unsigned)limbs * (n >> 12)), block(NTT_THREADS);
    const NttTables t = tables_of(ctx, inverse, limbs);
    const dim3 full(FULL_THREADS);
    if (n2 == 256 && !inverse) {
        launch_cols_fwd(data, src, d_src_rows, d_rows, d_mod_idx, t, n, limbs, st);
        launch_rows_fwd<false>(data, d_rows, d_mod_idx, t, n, limbs, FinishBatch(), st);
    } else if (!inverse) {
        hipLaunchKernelGGL(ntt_full_fwd<false>, grid, full, 0, st, data, src, d_src_rows, d_rows, d_mod_idx, t, n, FinishBatch());
    } else if (n2 == 256) {
        if (limbs <= SMALL_ROWS)
            hipLaunchKernelGGL(small_rows_inv, dim3(limbs * (n / SMALL_CHUNK)), dim3(SMALL_THREADS), 0, st, data, src, d_src_rows, d_rows,
                               d_mod_idx, t, n, (unsigned)g, fi);
        else
            hipLaunchKernelGGL(t.large && !fi.per ? ntt_rows256_inv<true> : ntt_rows256_inv<false>, grid, block, 0, st, data, src, d_src_rows, d_rows,
                               d_mod_idx, t, n, (unsigned)g, fi);
        if (limbs <= SMALL_COLS)
            hipLaunchKernelGGL(small_cols_inv, dim3(limbs * (256 / SMALL_CW)), dim3(64 * SMALL_CW), 0, st, data, d_rows, d_mod_idx, t, n);
        else hipLaunchKernelGGL(t.large ? ntt_cols_inv<true> : ntt_cols_inv<false>, grid, block, 0, st, data, d_rows, d_mod_idx, t, n, n2);
    } else {
        hipLaunchKernelGGL(ntt_full_inv, grid, full, 0, st, data, src, d_src_rows, d_rows, d_mod_idx, t, n, (unsigned)g, fi);
    }
}
// the second pass of an inverse transform whose row pass is done (launch_rows_ip)
void launch_cols_inv(cm_ctx *ctx, u64 *data, const int *d_rows, const int *d_mod_idx, int limbs, hipStream_t st) {
    if (limbs <= 0) return;
    Prof prof_(ctx, CM_K_NTT_INV, limbs, st);
    const int n = ctx->n;
    const NttTables t = tables_of(ctx, true, limbs);
    if (limbs <= SMALL_COLS)
        hipLaunchKernelGGL(small_cols_inv, dim3(limbs * (256 / SMALL_CW)), dim3(64 * SMALL_CW), 0, st, data, d_rows, d_mod_idx, t, n);
    else
        hipLaunchKernelGGL(t.large ? ntt_cols_inv<true> : ntt_cols_inv<false>, dim3(limbs * (n >> 12)), dim3(NTT_THREADS), 0, st, data, d_rows, d_mod_idx, t, n,
                           n >> 8);
}
void launch_mul_pt_rot_last_inv(cm_ctx *ctx, u64 *out, const MulPtBatch &b, int cnt, const u64 *pt_mont, int limbs, const int *d_mods, hipStream_t st) {
    if (ctx->n != 65536) {
        launch_mul_pt_rot_last(ctx, out, b, cnt, pt_mont, limbs, st);
        launch_ntt(ctx, out, d_mods, 2 * cnt, true, st);
        return;
    }
    {
        Prof prof_(ctx, CM_K_NTT_INV, 0, st);              // the limbs are counted with their second pass
        hipLaunchKernelGGL(small_rows_inv_mul, dim3(2 * cnt * (ctx->n / SMALL_CHUNK)), dim3(SMALL_THREADS), 0, st, out, b, pt_mont, limbs - 1, limbs,
                           tables_of(ctx, true, 2 * cnt), ctx->n);
    }
    launch_cols_inv(ctx, out, nullptr, d_mods, 2 * cnt, st);
}
void launch_ntt_fwd_finish(cm_ctx *ctx, u64 *conv, const int *d_mods, const FinishBatch &fb, hipStream_t st, const u64 *src,
                           const int *d_src_rows) {
    const int limbs = fb.items * fb.ncomp * (fb.level + 1), n = ctx->n;
    if (limbs <= 0) return;
    Prof prof_(ctx, CM_K_NTT_FWD, limbs, st);
    const NttTables t = tables_of(ctx, false, limbs);
    const int *none = nullptr;
    if (n == 4096) {
        hipLaunchKernelGGL(ntt_full_fwd<true>, dim3(limbs), dim3(FULL_THREADS), 0, st, conv, src, d_src_rows, none, d_mods, t, n, fb);
        return;
    }
    launch_cols_fwd(conv, src, d_src_rows, none, d_mods, t, n, limbs, st);
    launch_rows_fwd<true>(conv, none, d_mods, t, n, limbs, fb, st);
}
// Up to two workgroups a compute unit the repeated transforms are free; scores times V, eight relinearisations at a time, with 392, 800 and
// 1352 targets 302, 362 and 436 us joined, 322, 358 and 424 with the launch of its own.  More sources would be transformed one after the
// other.
#define JOIN_TARGETS 512
bool conv_joins_inv(const cm_ctx *ctx, bool near, int ns, int targets) { return ctx->n == 4096 && near && ns == 1 && targets <= JOIN_TARGETS; }
void launch_conv_ntt(cm_ctx *ctx, const ConvBatch &b, u64 *out, const u64 *in, hipStream_t st, const int *d_rows, const int *d_mods,
                     int limbs, const FinishBatch *fb) {
    const int n = ctx->n, ns = b.ns;              // rounded up to an instantiated bound below
    const NttTables t = tables_of(ctx, false, limbs);
    ConvArgs a;
    a.tabs = b.tabs, a.tab_step = b.tab_step, a.tab_period = b.tab_period ? b.tab_period : b.batch, a.in_group = b.in_group;
    a.in_stride = b.in_stride, a.out_stride = b.out_stride, a.own_stride = b.own_stride;
    a.own_src = b.own_src, a.own_g = b.own_g, a.nt = limbs >= CCF_NT;
    Prof prof_(ctx, CM_K_BASE_CONV, limbs, st);
    if (n == 4096) {
        const dim3 grid(b.max_nt + (b.own_src ? ns : 0), b.batch);
        const NttTables ti = tables_of(ctx, true, 0);
#define FULL_KERNEL(FB_, ...) hipLaunchKernelGGL((conv_full_fwd<__VA_ARGS__>), grid, dim3(FULL_THREADS), 0, st, out, in, a, t, ti, n, ctx->logn, FB_)
        if (b.inv) {
            if (fb) FULL_KERNEL(*fb, 1, true, false, true, true);
            else FULL_KERNEL(FinishBatch(), 1, false, false, true, true);
            return;
        }
#define FULL_FORM(NS_, NEAR_)                                                                                                    \
    do {                                                                                                                         \
        if (b.fold) FULL_KERNEL(*fb, NS_, true, true, NEAR_);                                                                    \
        else if (fb) FULL_KERNEL(*fb, NS_, true, false, NEAR_);                                                                  \
        else FULL_KERNEL(FinishBatch(), NS_, false, false, NEAR_);                                                               \
    } while (0)
#define FULL_LAUNCH(NS_)                                                                                                         \
    if (b.near) FULL_FORM(NS_, true);                                                                                            \
    else FULL_FORM(NS_, false)
        // the instantiation for eight spills 32 of 256 registers (27 with a tail, 59 with a folded limb) and still takes less than conversion
        // and transform in two launches (36 registers, no spills): a rotation on 16 + 8 primes, digits of eight, level 15, 69 -> 57 us;
        // five sources 66 -> 56
        if (ns <= 1) { FULL_LAUNCH(1); }
        else if (ns <= 2) { FULL_LAUNCH(2); }
        else if (ns <= 4) { FULL_LAUNCH(4); }
        else { FULL_FORM(8, false); }              // cut weights spill 40 to 70
#undef FULL_LAUNCH
#undef FULL_FORM
#undef FULL_KERNEL
        return;
    }
    a.tg = CCF_TG;
    while (a.tg > 1 && 256 / CCF_W * b.batch * ((b.max_nt + a.tg - 1) / a.tg) < CCF_FILL) a.tg >>= 1;
    a.groups = (b.max_nt + a.tg - 1) / a.tg;
    const dim3 grid(256 / CCF_W, a.groups + (b.own_src && !b.half ? 1 : 0), b.batch);
    // Eight sources spill twelve registers, 15 with cut weights (128 for two workgroups per compute unit), seven do not: with seven special
    // primes and digits of seven (14 + 7 primes, level 13) a rotation takes 129 us in the instantiation for eight and 116
    // in its own; 124 with conversion and column pass in two launches.  A raise and a ModDown each go by their own
    // count: eight special primes and digits of four, level 11, 128 us by the larger of the two, 116 by their own (123).
#define CCF_FORM(NS_, FOLD_)                                                                                                     \
    do {                                                                                                                         \
        if (b.near) hipLaunchKernelGGL((conv_cols_fwd<NS_, FOLD_, true>), grid, dim3(CCF_THREADS), 0, st, out, in, a, t, n, ctx->logn); \
        else hipLaunchKernelGGL((conv_cols_fwd<NS_, FOLD_, false>), grid, dim3(CCF_THREADS), 0, st, out, in, a, t, n, ctx->logn);  \
    } while (0)
#define CCF_LAUNCH(NS_)                                                                                                          \
    do {                                                                                                                         \
        if (b.fold) CCF_FORM(NS_, true);                                                                                         \
        else CCF_FORM(NS_, false);                                                                                               \
    } while (0)
    if (ns <= 1) CCF_LAUNCH(1);
    else if (ns <= 2) CCF_LAUNCH(2);
    else if (ns <= 4) CCF_LAUNCH(4);
    else if (ns <= 6) CCF_LAUNCH(6);
    else if (ns <= 7) CCF_FORM(7, false);   // never folded (ks_drop_fits)
    else CCF_LAUNCH(8);
#undef CCF_LAUNCH
#undef CCF_FORM
    if (b.half) return;
    if (fb) launch_rows_fwd<true>(out, d_rows, d_mods, t, n, limbs, *fb, st);
    else launch_rows_fwd<false>(out, d_rows, d_mods, t, n, limbs, FinishBatch(), st);
}
// a digit or a first component is a term of the sums (RipFp: 128 of them); an item of an integer limb holds eight
#define RIP_MAX_TERMS 120
#define RIP_SHARED_BETA 6          // draws of a wave: 2 KiB a digit, 64 KiB a workgroup
#define RIP_FILL 4096              // twice the waves that the chip holds at two a SIMD (8192 measured the same)
int rows_ip_items(int beta) { return RIP_MAX_TERMS / (beta + 1); }
// Integer ciphertext limbs (from 2^50 on): every wave of a sum of several items takes about the same long time, 256 of them a limb
// and output, and the chip holds RIP_WAVES_HELD at two a SIMD, so a launch takes whole rounds.  Where the last one is filled to less
// than 7/8, the row pass in a launch of its own is faster.  query times K (12 heads x 64, 17 key ciphertexts) with 58-bit primes and
// two special ones at level 7, 9 limbs, 1.1 rounds: 3320 us joined, 2940 apart; with 61-bit ones at level 2, 0.5 rounds: 1020 and 963;
// with six special primes at level 11, 2.1 rounds: 3920 and 3680; filled to 7/8 and more: level 13, 15 limbs, 6880 and 7120, embedding
// at level 4, 7 limbs, 98 and 103, with one special prime at level 6, 8 limbs, 143 and 157.  Single items and FP64 limbs (half the
// time a wave, more waves' worth of waiting to hide) are as fast or faster joined at every size measured.
#define RIP_WAVES_HELD 2048
bool rows_ip_fits(const cm_ctx *ctx, int beta, int level, int nz, int nsum) {
    if (ctx->n != 65536 || ctx->evk_stored_a || beta > 7 || nsum > rows_ip_items(beta)) return false;
    if (nsum == 1 || ctx->mod[level] < (1ULL << 50)) return true;
    const int waves = ctx->n / 256 * (level + 1 + ctx->K) * nz, rounds = (waves + RIP_WAVES_HELD - 1) / RIP_WAVES_HELD;
    return 8 * waves >= 7 * rounds * RIP_WAVES_HELD;
}
void launch_rows_ip(cm_ctx *ctx, const IpBatch &b, int beta, int level, hipStream_t st, int inv_from, const FoldIn &fi) {
    const int ext = level + 1 + ctx->K;
    Prof prof_(ctx, CM_K_INNER_PRODUCT, b.nz * b.nsum, st);
    RipArgs p;
    p.beta = beta, p.ext = ext, p.level = level, p.alpha = ctx->alpha, p.L = ctx->L, p.nmod = ctx->nmod, p.n = ctx->n, p.logn = ctx->logn;
    p.kdig = (ctx->L + ctx->alpha) / ctx->alpha, p.inv_from = inv_from, p.ubound = ctx->d_ubound, p.pmont = ctx->d_pmont;
    const NttTables t = tables_of(ctx, false, 0), ti = tables_of(ctx, true, 0);
    bool shared = b.nz > 1 && b.nsum == 1 && beta <= RIP_SHARED_BETA;
    for (int z = 0; z < b.nz; z++) shared = shared && b.it[z].key == b.it[0].key && !b.it[z].g;
    if (shared) {
        // runs as long as they leave RIP_FILL waves
        int per = b.nz;
        while (per > 1 && ctx->n / 256 * ext * ((b.nz + per - 1) / per) < RIP_FILL) per = (per + 1) / 2;
        hipLaunchKernelGGL(k_rows_ip<true>, dim3(ctx->n / (256 * RIP_WAVES), ext, (b.nz + per - 1) / per), dim3(64 * RIP_WAVES),
                           RIP_WAVES * (RIP_ROW + 256 * beta) * 8, st, b, p, fi, t, ti, per);
        return;
    }
    hipLaunchKernelGGL(k_rows_ip<false>, dim3(ctx->n / (256 * RIP_WAVES), ext, b.nz), dim3(64 * RIP_WAVES), RIP_WAVES * RIP_ROW * 8, st, b, p, fi, t,
                       ti, 1);
}
void launch_ntt_rows(cm_ctx *ctx, u64 *data, const int *d_rows, const int *d_mod_idx, int limbs,
                     bool inverse, hipStream_t st) {
    launch_ntt_src(ctx, data, d_rows, nullptr, nullptr, d_mod_idx, limbs, inverse, st, 0);
}
void launch_ntt(cm_ctx *ctx, u64 *data, const int *d_mod_idx, int limbs, bool inverse,
                hipStream_t st) {
    launch_ntt_rows(ctx, data, nullptr, d_mod_idx, limbs, inverse, st);
}
void launch_ntt_range(cm_ctx *ctx, u64 *data, int first_mod, int limbs, bool inverse,
                      hipStream_t st) {
    launch_ntt(ctx, data, iota_idx(ctx) + first_mod, limbs, inverse, st);
}
