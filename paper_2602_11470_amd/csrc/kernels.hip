// Element-wise, base-conversion, key-switch and sampling kernels of libcachemir (gfx950).
// Polynomials are [limbs][n] 64-bit words.  "mont" operands are pre-multiplied by 2^64 mod q.
#include "kernels.h"

#define TPB 256
typedef u64 u64x2 __attribute__((ext_vector_type(2)));


// ---- a short list of integers into device memory without a copy or an allocation ---------------
// (the values travel as kernel arguments, so the launch can be captured into a graph)
#define IDX_CHUNK 256
struct IdxChunk { int v[IDX_CHUNK]; };
__global__ void k_set_idx(int *dst, IdxChunk c, int count) {
    const int i = threadIdx.x;
    if (i < count) dst[i] = c.v[i];
}
void launch_set_idx(int *d_dst, const int *h_src, int count, hipStream_t st) {
    for (int base = 0; base < count; base += IDX_CHUNK) {
        IdxChunk c;
        const int m = count - base < IDX_CHUNK ? count - base : IDX_CHUNK;
        for (int i = 0; i < IDX_CHUNK; i++) c.v[i] = i < m ? h_src[base + i] : 0;
        hipLaunchKernelGGL(k_set_idx, dim3(1), dim3(IDX_CHUNK), 0, st, d_dst + base, c, m);
    }
}

// ---- signed integers -> residues -------------------------------------------------------------
__global__ void k_reduce_i64(u64 *out, const long long *coeffs, const int *mod_idx, const ModC *modc, int n) {
    int i = blockIdx.x * TPB + threadIdx.x, l = blockIdx.y;
    const ModC m = modc[mod_idx[l]];
    long long c = coeffs[i];
    u64 a = c < 0 ? (u64)(-(c + 1)) + 1ULL : (u64)c;        // |c| without overflow
    u64 r = redc((u128)to_mont(a, m), m.q, m.qinv);         // |c| mod q
    out[(size_t)l * n + i] = (c < 0 && r) ? m.q - r : r;
}
void launch_reduce_i64(cm_ctx *ctx, u64 *out, const long long *d_coeffs, const int *d_mod_idx, int limbs, hipStream_t st) {
    hipLaunchKernelGGL(k_reduce_i64, dim3(ctx->n / TPB, limbs), dim3(TPB), 0, st, out, d_coeffs, d_mod_idx, ctx->d_modc, ctx->n);
}

__global__ void k_to_mont(u64 *data, const int *mod_idx, const ModC *modc, int n) {
    int i = blockIdx.x * TPB + threadIdx.x, l = blockIdx.y;
    const ModC m = modc[mod_idx[l]];
    size_t o = (size_t)l * n + i;
    data[o] = to_mont(data[o], m);
}
void launch_to_mont(cm_ctx *ctx, u64 *data, const int *d_mod_idx, int limbs, hipStream_t st) {
    hipLaunchKernelGGL(k_to_mont, dim3(ctx->n / TPB, limbs), dim3(TPB), 0, st, data, d_mod_idx, ctx->d_modc, ctx->n);
}
__global__ void k_from_mont(u64 *out, const u64 *in, const int *mod_idx, const ModC *modc, int n) {
    int i = blockIdx.x * TPB + threadIdx.x, l = blockIdx.y;
    const ModC m = modc[mod_idx[l]];
    size_t o = (size_t)l * n + i;
    out[o] = redc((u128)in[o], m.q, m.qinv);
}
void launch_from_mont(cm_ctx *ctx, u64 *out, const u64 *in, const int *d_mod_idx, int limbs, hipStream_t st) {
    hipLaunchKernelGGL(k_from_mont, dim3(ctx->n / TPB, limbs), dim3(TPB), 0, st, out, in, d_mod_idx, ctx->d_modc, ctx->n);
}

// ---- ciphertext element-wise ---------------------------------------------------------------------
// rows = ncomp*limbs; row r has modulus index r % limbs
__global__ void k_add(u64 *out, const u64 *a, const u64 *b, const ModC *modc, int limbs, int n) {
    int i = blockIdx.x * TPB + threadIdx.x, r = blockIdx.y;
    u64 q = modc[r % limbs].q;
    size_t o = (size_t)r * n + i;
    out[o] = addmod(a[o], b[o], q);
}
void launch_add(cm_ctx *ctx, u64 *out, const u64 *a, const u64 *b, int ncomp, int limbs, hipStream_t st) {
    Prof prof_(ctx, CM_K_ELEMENTWISE, ncomp * limbs, st);
    hipLaunchKernelGGL(k_add, dim3(ctx->n / TPB, ncomp * limbs), dim3(TPB), 0, st, out, a, b, ctx->d_modc, limbs, ctx->n);
}

__global__ void k_mul_pt(u64 *out, const u64 *a, const u64 *pt_mont, const ModC *modc, int limbs, int n) {
    int i = blockIdx.x * TPB + threadIdx.x, r = blockIdx.y;
    const ModC m = modc[r % limbs];
    size_t o = (size_t)r * n + i;
    out[o] = redc((u128)a[o] * pt_mont[(size_t)(r % limbs) * n + i], m.q, m.qinv);
}
void launch_mul_pt(cm_ctx *ctx, u64 *out, const u64 *a, const u64 *pt_mont, int ncomp, int limbs, hipStream_t st) {
    Prof prof_(ctx, CM_K_ELEMENTWISE, ncomp * limbs, st);
    hipLaunchKernelGGL(k_mul_pt, dim3(ctx->n / TPB, ncomp * limbs), dim3(TPB), 0, st, out, a, pt_mont, ctx->d_modc, limbs, ctx->n);
}

// out[z][2][limbs][n] = src_z * perm_{g_z}(pt): up to CM_MASK_BATCH ciphertexts times slot rotations of one
// plaintext (the rotation is the Galois permutation of its evaluation-domain words), one launch
__global__ void k_mul_pt_rot_batch(u64 *__restrict__ out, MulPtBatch b, const u64 *__restrict__ pt_mont,
                                   const ModC *__restrict__ modc, int limbs, int n, int logn) {
    const unsigned i = blockIdx.x * TPB + threadIdx.x;
    const int r = blockIdx.y, z = blockIdx.z, l = r % limbs;
    const ModC m = modc[l];
    const unsigned g = b.g[z];
    const unsigned s = g ? perm_src(i, g, logn) : i;
    out[((size_t)z * 2 * limbs + r) * n + i] = redc((u128)b.src[z][(size_t)r * n + i] * pt_mont[(size_t)l * n + s], m.q, m.qinv);
}
__global__ void k_mul_pt_rot_last(u64 *__restrict__ out, MulPtBatch b, const u64 *__restrict__ pt_mont,
                                  const ModC *__restrict__ modc, int limbs, int n, int logn) {
    const unsigned i = blockIdx.x * TPB + threadIdx.x;
    const int c = blockIdx.y, z = blockIdx.z, l = limbs - 1;
    const ModC m = modc[l];
    const unsigned g = b.g[z];
    const unsigned s = g ? perm_src(i, g, logn) : i;
    out[((size_t)z * 2 + c) * n + i] = redc((u128)b.src[z][((size_t)c * limbs + l) * n + i] * pt_mont[(size_t)l * n + s], m.q, m.qinv);
}
void launch_mul_pt_rot_last(cm_ctx *ctx, u64 *out, const MulPtBatch &b, int cnt, const u64 *pt_mont, int limbs, hipStream_t st) {
    Prof prof_(ctx, CM_K_ELEMENTWISE, cnt * 2, st);
    hipLaunchKernelGGL(k_mul_pt_rot_last, dim3(ctx->n / TPB, 2, cnt), dim3(TPB), 0, st, out, b, pt_mont, ctx->d_modc, limbs, ctx->n,
                       ctx->logn);
}
// the same with ONE source for all cnt products: its word is read once and the lane walks over the rotations
__global__ void k_mul_pt_rot_same(u64 *__restrict__ out, MulPtBatch b, int cnt, const u64 *__restrict__ pt_mont,
                                  const ModC *__restrict__ modc, int limbs, int n, int logn) {
    const unsigned i = blockIdx.x * TPB + threadIdx.x;
    const int r = blockIdx.y, l = r % limbs;
    const ModC m = modc[l];
    const u64 v = b.src[0][(size_t)r * n + i];
    for (int z = 0; z < cnt; z++) {
        const unsigned g = b.g[z];
        const unsigned s = g ? perm_src(i, g, logn) : i;
        out[((size_t)z * 2 * limbs + r) * n + i] = redc((u128)v * pt_mont[(size_t)l * n + s], m.q, m.qinv);
    }
}
void launch_mul_pt_rot_batch(cm_ctx *ctx, u64 *out, const MulPtBatch &b, int cnt, const u64 *pt_mont, int limbs, hipStream_t st) {
    Prof prof_(ctx, CM_K_ELEMENTWISE, cnt * 2 * limbs, st);
    bool same = cnt > 1;
    for (int z = 1; z < cnt; z++) same = same && b.src[z] == b.src[0];
    if (same) {
        hipLaunchKernelGGL(k_mul_pt_rot_same, dim3(ctx->n / TPB, 2 * limbs), dim3(TPB), 0, st, out, b, cnt, pt_mont, ctx->d_modc,
                           limbs, ctx->n, ctx->logn);
        return;
    }
    hipLaunchKernelGGL(k_mul_pt_rot_batch, dim3(ctx->n / TPB, 2 * limbs, cnt), dim3(TPB), 0, st, out, b, pt_mont, ctx->d_modc,
                       limbs, ctx->n, ctx->logn);
}

// acc (+)= a * pt_mont over ncomp components; accumulate != 0 adds into out
__global__ void k_mac_pt(u64 *out, const u64 *a, const u64 *pt_mont, const ModC *modc, int limbs, int n, int accumulate) {
    int i = blockIdx.x * TPB + threadIdx.x, r = blockIdx.y;
    const ModC m = modc[r % limbs];
    size_t o = (size_t)r * n + i;
    u64 v = redc((u128)a[o] * pt_mont[(size_t)(r % limbs) * n + i], m.q, m.qinv);
    out[o] = accumulate ? addmod(out[o], v, m.q) : v;
}
void launch_mac_pt(cm_ctx *ctx, u64 *out, const u64 *a, const u64 *pt_mont, int ncomp, int limbs, int accumulate, hipStream_t st) {
    Prof prof_(ctx, CM_K_ELEMENTWISE, ncomp * limbs, st);
    hipLaunchKernelGGL(k_mac_pt, dim3(ctx->n / TPB, ncomp * limbs), dim3(TPB), 0, st, out, a, pt_mont, ctx->d_modc, limbs, ctx->n, accumulate);
}

// Tensor product of two 2-component ciphertexts: (a0 b0, a0 b1 + a1 b0, a1 b1); accumulate adds.
__global__ void k_tensor(u64 *out, const u64 *a, const u64 *b, const ModC *modc, int limbs, int n, int accumulate) {
    int i = blockIdx.x * TPB + threadIdx.x, l = blockIdx.y;
    const ModC m = modc[l];
    size_t o = (size_t)l * n + i, cs = (size_t)limbs * n;
    u64 a0 = to_mont(a[o], m), a1 = to_mont(a[o + cs], m);
    u64 b0 = b[o], b1 = b[o + cs];
    u64 d0 = redc((u128)a0 * b0, m.q, m.qinv);
    u64 d1 = redc((u128)a0 * b1 + (u128)a1 * b0, m.q, m.qinv);     // two products: (T >> 64) < q holds for q < 2^63
    u64 d2 = redc((u128)a1 * b1, m.q, m.qinv);
    if (accumulate) {
        d0 = addmod(d0, out[o], m.q);
        d1 = addmod(d1, out[o + cs], m.q);
        d2 = addmod(d2, out[o + 2 * cs], m.q);
    }
    out[o] = d0;
    out[o + cs] = d1;
    out[o + 2 * cs] = d2;
}
// out[z][3][limbs][n] = a (x) b[z] for cnt ciphertexts b stacked at stride 2*limbs*n: one launch
__global__ void k_tensor_batch(u64 *__restrict__ out, const u64 *__restrict__ a, const u64 *__restrict__ b,
                               const ModC *__restrict__ modc, int limbs, int n) {
    int i = blockIdx.x * TPB + threadIdx.x, l = blockIdx.y, z = blockIdx.z;
    const ModC m = modc[l];
    size_t o = (size_t)l * n + i, cs = (size_t)limbs * n;
    u64 a0 = to_mont(a[o], m), a1 = to_mont(a[o + cs], m);
    const u64 *bz = b + (size_t)z * 2 * cs;
    u64 *oz = out + (size_t)z * 3 * cs;
    u64 b0 = bz[o], b1 = bz[o + cs];
    oz[o] = redc((u128)a0 * b0, m.q, m.qinv);
    oz[o + cs] = redc((u128)a0 * b1 + (u128)a1 * b0, m.q, m.qinv);
    oz[o + 2 * cs] = redc((u128)a1 * b1, m.q, m.qinv);
}
void launch_tensor_batch(cm_ctx *ctx, u64 *out, const u64 *a, const u64 *b, int cnt, int limbs, hipStream_t st) {
    Prof prof_(ctx, CM_K_ELEMENTWISE, 3 * limbs * cnt, st);
    hipLaunchKernelGGL(k_tensor_batch, dim3(ctx->n / TPB, limbs, cnt), dim3(TPB), 0, st, out, a, b, ctx->d_modc, limbs, ctx->n);
}
// acc[2][limbs][n] (+)= sum_z src[z] * (pt rotated by g[z]); src stacked at stride 2*limbs*n: one launch, acc written once
__global__ void k_mac_pt_rot_batch(u64 *acc, const u64 *__restrict__ src, MulPtBatch b, int cnt,
                                   const u64 *__restrict__ pt_mont, const ModC *__restrict__ modc, int limbs, int n, int logn,
                                   int accumulate) {
    const unsigned i = blockIdx.x * TPB + threadIdx.x;
    const int r = blockIdx.y, l = r % limbs;
    const ModC m = modc[l];
    const size_t o = (size_t)r * n + i;
    u64 v = accumulate ? acc[o] : 0;
    for (int z = 0; z < cnt; z++) {
        const unsigned g = b.g[z];
        const unsigned s = g ? perm_src(i, g, logn) : i;
        v = addmod(v, redc((u128)src[(size_t)z * 2 * limbs * n + o] * pt_mont[(size_t)l * n + s], m.q, m.qinv), m.q);
    }
    acc[o] = v;
}
void launch_mac_pt_rot_batch(cm_ctx *ctx, u64 *acc, const u64 *src, const MulPtBatch &b, int cnt, const u64 *pt_mont,
                             int limbs, int accumulate, hipStream_t st) {
    Prof prof_(ctx, CM_K_ELEMENTWISE, cnt * 2 * limbs, st);
    hipLaunchKernelGGL(k_mac_pt_rot_batch, dim3(ctx->n / TPB, 2 * limbs), dim3(TPB), 0, st, acc, src, b, cnt, pt_mont,
                       ctx->d_modc, limbs, ctx->n, ctx->logn, accumulate);
}
// FP64 modular products for limbs whose modulus is below 2^50: residues as exact integers in doubles, a product
//     h = y a;  l = fma(y, a, -h);  c = rint(y (a / q));  r = fma(-c, q, h) + l        (|r| < q)
// with a / q taken as a * (1 / q); four terms may be summed before a sum is renormalised (|sum| < 4.6 q < 2^53 stays exact)
struct MacFp {
    double q, qinv;
    __device__ __forceinline__ double mulmod(double y, double a, double aq) const {
        double h = y * a;
        double l = __builtin_fma(y, a, -h);
        double c = __builtin_rint(y * aq);
        return __builtin_fma(-c, q, h) + l;
    }
    __device__ __forceinline__ double norm(double x) const { return __builtin_fma(-__builtin_rint(x * qinv), q, x); }
    __device__ __forceinline__ static double from_u64(u64 raw) {                 // raw < 2^52
        return __longlong_as_double((long long)(raw | 0x4330000000000000ULL)) - 4503599627370496.0;
    }
    __device__ __forceinline__ u64 canon(double v) const {                       // |v| < 2^53 -> [0, q)
        const double r = norm(v);                                                // |r| < q: q is added under the sign mask
        const int m = __double2hiint(r) >> 31;
        const double a = __hiloint2double(__double2hiint(q) & m, __double2loint(q) & m);
        return (u64)__double_as_longlong((r + a) + 4503599627370496.0) & 0x000FFFFFFFFFFFFFULL;
    }
};
// out[z][3][limbs][n] = sum_{j < cnt} a[j] (x) b[z*gs + j*ts]: a and b stacked at stride 2*limbs*n (gs, ts = the distance of
// groups and of the terms of a group in b, in ciphertexts); every output written once.
// On limbs below 2^50 the four products per term run in FP64 (no multiplier form needed), sums renormalised every two terms.
__global__ void k_tensor_sum(u64 *__restrict__ out, const u64 *__restrict__ a, const u64 *__restrict__ b,
                             const ModC *__restrict__ modc, const FpQ *__restrict__ fpq, int limbs, int n, int cnt, int gs,
                             int ts) {
    int i = blockIdx.x * TPB + threadIdx.x, l = blockIdx.y, z = blockIdx.z;
    const ModC m = modc[l];
    const size_t o = (size_t)l * n + i, cs = (size_t)limbs * n;
    const FpQ fq = fpq[l];
    if (fq.q != 0.0) {
        const MacFp F{fq.q, fq.qinv};
        double d0 = 0.0, d1 = 0.0, d2 = 0.0;
        for (int j = 0; j < cnt; j++) {
            const u64 *aj = a + (size_t)j * 2 * cs, *bj = b + ((size_t)z * gs + (size_t)j * ts) * 2 * cs;
            const double a0 = MacFp::from_u64(aj[o]), a1 = MacFp::from_u64(aj[o + cs]);
            const double b0 = MacFp::from_u64(__builtin_nontemporal_load(bj + o));
            const double b1 = MacFp::from_u64(__builtin_nontemporal_load(bj + o + cs));
            const double b0q = b0 * F.qinv, b1q = b1 * F.qinv;
            d0 += F.mulmod(a0, b0, b0q);
            d1 += F.mulmod(a0, b1, b1q) + F.mulmod(a1, b0, b0q);
            d2 += F.mulmod(a1, b1, b1q);
            if (j & 1) d0 = F.norm(d0), d1 = F.norm(d1), d2 = F.norm(d2);
        }
        u64 *oz = out + (size_t)z * 3 * cs;
        oz[o] = F.canon(d0);
        oz[o + cs] = F.canon(d1);
        oz[o + 2 * cs] = F.canon(d2);
        return;
    }
    u64 d0 = 0, d1 = 0, d2 = 0;
    for (int j = 0; j < cnt; j++) {
        const u64 *aj = a + (size_t)j * 2 * cs, *bj = b + ((size_t)z * gs + (size_t)j * ts) * 2 * cs;
        const u64 a0 = to_mont(aj[o], m), a1 = to_mont(aj[o + cs], m);
        const u64 b0 = __builtin_nontemporal_load(bj + o), b1 = __builtin_nontemporal_load(bj + o + cs);
        d0 = addmod(d0, redc((u128)a0 * b0, m.q, m.qinv), m.q);
        d1 = addmod(d1, redc((u128)a0 * b1 + (u128)a1 * b0, m.q, m.qinv), m.q);
        d2 = addmod(d2, redc((u128)a1 * b1, m.q, m.qinv), m.q);
    }
    u64 *oz = out + (size_t)z * 3 * cs;
    oz[o] = d0;
    oz[o + cs] = d1;
    oz[o + 2 * cs] = d2;
}
// The same sums with the cnt <= TS_MAX_CNT ciphertexts a[j] held in registers (FP64 limbs only) while the lane runs over
// all groups: a is read once instead of once per group, which is half of the traffic when a does not fit the caches.
// HELD: stores in a stream of reads cost more than their bytes (k_vmm_mac); the sums wait in LDS (48 KiB for eight groups: TS_HELD
// workgroups a compute unit) and a launch is the limbs whose workgroups are there at once, which all write at its end.  Against one
// launch that writes group by group: 128 ciphertexts at level 22 736 -> 666 us, at level 3 120 -> 112; scores times V at level 22 3650 ->
// 3590.  Which of the two a sum takes: tensor_sum_held.
#define TS_MAX_CNT 16
#define TS_MAX_GROUPS 8
#define TS_HELD 3
template <bool HELD>
__global__ __launch_bounds__(TPB, HELD ? TS_HELD : 1) void k_tensor_sum_stationary(u64 *__restrict__ out, const u64 *__restrict__ a,
                                                               const u64 *__restrict__ b, const FpQ *__restrict__ fpq,
                                                               int limbs, int n, int cnt, int groups, int gs, int ts, int l0) {
    extern __shared__ u64 ts_sums[];
    const int i = blockIdx.x * TPB + threadIdx.x, l = l0 + blockIdx.y;
    const FpQ fq = fpq[l];
    const MacFp F{fq.q, fq.qinv};
    const size_t o = (size_t)l * n + i, cs = (size_t)limbs * n;
    double a0[TS_MAX_CNT], a1[TS_MAX_CNT];
#pragma unroll
    for (int j = 0; j < TS_MAX_CNT; j++) {
        a0[j] = j < cnt ? MacFp::from_u64(a[(size_t)j * 2 * cs + o]) : 0.0;
        a1[j] = j < cnt ? MacFp::from_u64(a[(size_t)j * 2 * cs + cs + o]) : 0.0;
    }
    for (int z = 0; z < groups; z++) {
        double d0 = 0.0, d1 = 0.0, d2 = 0.0;
        // Eight terms at a time: their sixteen words are requested before the first is used.  Terms at or past cnt read
        // term 0's words again (a valid address) and multiply them by a zero, so no load sits behind a branch.
#pragma unroll
        for (int jc = 0; jc < TS_MAX_CNT; jc += 8) {
            if (jc < cnt) {
                u64 r0[8], r1[8];
#pragma unroll
                for (int jj = 0; jj < 8; jj++) {
                    const int j = jc + jj < cnt ? jc + jj : 0;
                    const u64 *bj = b + ((size_t)z * gs + (size_t)j * ts) * 2 * cs;
                    r0[jj] = __builtin_nontemporal_load(bj + o), r1[jj] = __builtin_nontemporal_load(bj + o + cs);
                }
#pragma unroll
                for (int jj = 0; jj < 8; jj++) {
                    const int j = jc + jj;
                    const double b0 = MacFp::from_u64(r0[jj]), b1 = MacFp::from_u64(r1[jj]);
                    const double b0q = b0 * F.qinv, b1q = b1 * F.qinv;
                    d0 += F.mulmod(a0[j], b0, b0q);
                    d1 += F.mulmod(a0[j], b1, b1q) + F.mulmod(a1[j], b0, b0q);
                    d2 += F.mulmod(a1[j], b1, b1q);
                    if (jj & 1) d0 = F.norm(d0), d1 = F.norm(d1), d2 = F.norm(d2);
                }
            }
        }
        u64 *w = HELD ? ts_sums + z * (3 * TPB) + threadIdx.x : out + (size_t)z * 3 * cs + o;
        const size_t ws = HELD ? TPB : cs;
        w[0] = F.canon(d0);
        w[ws] = F.canon(d1);
        w[2 * ws] = F.canon(d2);
    }
    if (HELD) {
        for (int r = 0; r < 3 * groups; r++) out[r * cs + o] = ts_sums[r * TPB + threadIdx.x];
    }
}
static int ts_launch_limbs(int n) { return std::max(1, 256 * TS_HELD * TPB / n); }
// A launch that ends before the next begins pays for its start and its last wave: short ones (few terms), many of them, and launches
// that do not fill the chip lose more than the writes cost.  Held against written as they come, (cnt, groups), three limbs to a launch at
// n = 65536: one launch always gains (3 limbs (1, 2) 10.6 us, 11.7; (16, 8) 77, 90; n = 4096, 8 limbs 6.0, 7.0 and 25.7, 41); two launches
// that are full (6 limbs) from (2, 4) on: 34.3, 38.1; 4 limbs (16, 2) 40.9, 39.2; (16, 4) 64.8, 65.2; (4, 8) 47.2, 44.5; 10 limbs (8, 8)
// 150, 160; (8, 4) 86, 89; (8, 2) 56.2, 53.9; (2, 8) 105, 99; 21 limbs (16, 2) 211, 230; (8, 4) 189, 199; (8, 2) 109.5, 106.8; (1, 2) 74, 60.
bool tensor_sum_held(int n, int limbs, int cnt, int groups) {
    const int per = ts_launch_limbs(n), launches = (limbs + per - 1) / per, terms = cnt * groups;
    if (launches == 1 || terms >= 64) return true;
    return 4 * limbs >= 3 * launches * per && terms >= (launches == 2 ? 8 : 32);
}
// The same sums for PASSES sets of ciphertexts a against one b: out[pass] and a[pass] stacked at out_pass and a_pass words.  A wave
// owns a pass for 64 coefficients; the words of a group are staged in LDS for all of them, the next group's requested ahead.
// Bound by HBM: with a launch a pass the cache was read once per pass of a grouped query.  Four passes over 128 ciphertexts of ten
// limbs 4 x 317 -> 582 us, grouped-query attention at level 9 12860 -> 11640.  108 registers because the
// terms are worked on four at a time (sched_barrier); left to itself the compiler spills 187 of 128.
#define TS_CO 64
template <int PASSES>
__global__ __launch_bounds__(64 * PASSES, 4) void k_tensor_sum_passes(u64 *__restrict__ out, const u64 *__restrict__ a, const u64 *__restrict__ b,
                                                                   const FpQ *__restrict__ fpq, int limbs, int n, int cnt, int groups, int gs, int ts,
                                                                   size_t out_pass, size_t a_pass) {
    constexpr int ROWS = 2 * TS_MAX_CNT / PASSES;
    __shared__ double sb[2][2 * TS_MAX_CNT * TS_CO];
    const int co = threadIdx.x & 63, pass = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = blockIdx.y;
    const FpQ fq = fpq[l];
    const MacFp F{fq.q, fq.qinv};
    const size_t o = (size_t)l * n + blockIdx.x * TS_CO + co, cs = (size_t)limbs * n;
    a += pass * a_pass, out += pass * out_pass;
    u64 r[ROWS];
    // row = 2 j + component; rows of terms at or past cnt hold the last term's words again, and multiply zeros
    auto request = [&](int z) {
#pragma unroll
        for (int it = 0; it < ROWS; it++) {
            const int row = pass * ROWS + it, j = min(row >> 1, cnt - 1);
            r[it] = __builtin_nontemporal_load(b + (((size_t)z * gs + (size_t)j * ts) * 2 + (row & 1)) * cs + o);
        }
    };
    request(0);
    double a0[TS_MAX_CNT], a1[TS_MAX_CNT];
#pragma unroll
    for (int j = 0; j < TS_MAX_CNT; j++) {
        a0[j] = j < cnt ? MacFp::from_u64(a[(size_t)j * 2 * cs + o]) : 0.0;
        a1[j] = j < cnt ? MacFp::from_u64(a[(size_t)j * 2 * cs + cs + o]) : 0.0;
    }
    for (int z = 0; z < groups; z++) {
        // two buffers in turn: a wave that writes to one has passed the barrier behind the others' reads of it
        double *s = sb[z & 1] + co;
#pragma unroll
        for (int it = 0; it < ROWS; it++) s[(pass * ROWS + it) * TS_CO] = MacFp::from_u64(r[it]);
        __syncthreads();
        if (z + 1 < groups) request(z + 1);
        double d0 = 0.0, d1 = 0.0, d2 = 0.0;
#pragma unroll
        for (int j = 0; j < TS_MAX_CNT; j++) {
            const double b0 = s[2 * j * TS_CO], b1 = s[(2 * j + 1) * TS_CO], b0q = b0 * F.qinv, b1q = b1 * F.qinv;
            d0 += F.mulmod(a0[j], b0, b0q);
            d1 += F.mulmod(a0[j], b1, b1q) + F.mulmod(a1[j], b0, b0q);
            d2 += F.mulmod(a1[j], b1, b1q);
            if (j & 1) d0 = F.norm(d0), d1 = F.norm(d1), d2 = F.norm(d2);
            if ((j & 3) == 3) __builtin_amdgcn_sched_barrier(0);
        }
        u64 *oz = out + (size_t)z * 3 * cs;
        oz[o] = F.canon(d0);
        oz[o + cs] = F.canon(d1);
        oz[o + 2 * cs] = F.canon(d2);
    }
}
// Where the joint launch is the faster way.  It always does the work of TS_MAX_CNT terms and its writes lie among its reads: with few
// terms, and two passes with few groups, a launch a pass takes less.  Ten limbs at n = 65536, (cnt, groups), joint against single: two
// passes (16, 8) 464 us, 565; (16, 4) 310, 330; (16, 1) 200, 132; (8, 8) 358, 316; (1, 2) 87, 63; four passes (16, 8) 585, 1129;
// (16, 1) 234, 265; (8, 1) 141, 146 (13 limbs: 180, 179); (4, 1) 78, 70; (1, 2) 104, 127; (2, 4) 208, 235; (2, 8) 398, 407 (21 limbs: 818, 790).
// A launch that the chip holds at once (n = 4096) is bound by its own latency, and calls of it are faster joint or equal: 8 limbs, four
// passes 6 to 36 us joint, 16 to 110 single, two passes 6.5 to 32 against 8.5 to 51; grouped-query attention at level 3 with two passes over
// (2, 8), (1, 8) and (4, 4) 912, 847 and 810 us against 938, 866 and 825, with 13 limbs within 0.3 % of each other.
bool tensor_sum_passes_pays(int n, int limbs, int cnt, int groups, int passes) {
    if (n / TS_CO * limbs <= 1024) return true;
    if (passes == 2) return cnt >= 16 && groups >= 4;
    return groups == 1 ? cnt >= 16 : cnt >= 4 || groups <= 4;
}
bool tensor_sum_passes_fits(const cm_ctx *ctx, int cnt, int groups, int limbs, int passes) {
    if ((passes != 2 && passes != TS_PASSES) || cnt > TS_MAX_CNT) return false;
    for (int l = 0; l < limbs; l++)
        if (ctx->mod[l] >= (1ULL << 50)) return false;
    return tensor_sum_passes_pays(ctx->n, limbs, cnt, groups, passes);
}
void launch_tensor_sum_passes(cm_ctx *ctx, u64 *out, size_t out_pass, const u64 *a, size_t a_pass, int passes, const u64 *b, int cnt, int groups,
                              int limbs, hipStream_t st, int gs, int ts) {
    Prof prof_(ctx, CM_K_ELEMENTWISE, 3 * limbs * groups * passes, st);
    const dim3 grid(ctx->n / TS_CO, limbs);
    if (passes == 2)
        hipLaunchKernelGGL(k_tensor_sum_passes<2>, grid, dim3(128), 0, st, out, a, b, ctx->d_fpq, limbs, ctx->n, cnt, groups, gs, ts, out_pass, a_pass);
    else
        hipLaunchKernelGGL(k_tensor_sum_passes<TS_PASSES>, grid, dim3(64 * TS_PASSES), 0, st, out, a, b, ctx->d_fpq, limbs, ctx->n, cnt, groups, gs, ts,
                           out_pass, a_pass);
}
void launch_tensor_sum(cm_ctx *ctx, u64 *out, const u64 *a, const u64 *b, int cnt, int groups, int limbs, hipStream_t st,
                       int group_stride, int term_stride) {
    const int gs = group_stride ? group_stride : cnt, ts = term_stride ? term_stride : 1;
    Prof prof_(ctx, CM_K_ELEMENTWISE, 3 * limbs * groups, st);
    bool all_fp = true;
    for (int l = 0; l < limbs; l++) all_fp = all_fp && ctx->mod[l] < (1ULL << 50);
    if (all_fp && cnt <= TS_MAX_CNT && groups > 1 && groups <= TS_MAX_GROUPS) {
        if (!tensor_sum_held(ctx->n, limbs, cnt, groups)) {
            hipLaunchKernelGGL(k_tensor_sum_stationary<false>, dim3(ctx->n / TPB, limbs), dim3(TPB), 0, st, out, a, b, ctx->d_fpq, limbs, ctx->n, cnt,
                               groups, gs, ts, 0);
            return;
        }
        const int per = ts_launch_limbs(ctx->n), launches = (limbs + per - 1) / per;
        for (int i = 0; i < launches; i++) {
            const int l0 = limbs * i / launches, l1 = limbs * (i + 1) / launches;
            hipLaunchKernelGGL(k_tensor_sum_stationary<true>, dim3(ctx->n / TPB, l1 - l0), dim3(TPB), groups * 3 * TPB * 8, st, out, a, b, ctx->d_fpq, limbs,
                               ctx->n, cnt, groups, gs, ts, l0);
        }
        return;
    }
    hipLaunchKernelGGL(k_tensor_sum, dim3(ctx->n / TPB, limbs, groups), dim3(TPB), 0, st, out, a, b, ctx->d_modc, ctx->d_fpq, limbs, ctx->n,
                       cnt, gs, ts);
}
void launch_tensor(cm_ctx *ctx, u64 *out, const u64 *a, const u64 *b, int limbs, int accumulate, hipStream_t st) {
    Prof prof_(ctx, CM_K_ELEMENTWISE, 3 * limbs, st);
    hipLaunchKernelGGL(k_tensor, dim3(ctx->n / TPB, limbs), dim3(TPB), 0, st, out, a, b, ctx->d_modc, limbs, ctx->n, accumulate);
}

// Galois map on evaluation-domain rows (a pure permutation); rows = ncomp*limbs
__global__ void k_automorphism(u64 *out, const u64 *in, int n, int logn, unsigned g) {
    unsigned i = blockIdx.x * TPB + threadIdx.x;
    size_t r = blockIdx.y;
    out[r * n + i] = in[r * n + perm_src(i, g, logn)];
}
void launch_automorphism(cm_ctx *ctx, u64 *out, const u64 *in, int rows, u64 g, hipStream_t st) {
    Prof prof_(ctx, CM_K_ELEMENTWISE, rows, st);
    hipLaunchKernelGGL(k_automorphism, dim3(ctx->n / TPB, rows), dim3(TPB), 0, st, out, in, ctx->n, ctx->logn, (unsigned)g);
}

// ---- evaluation-key inner product ------------------------------------------------------------------
// u0[r] = sum_j dig[j][r] * evk[j][0][mod(r)],  u1 likewise with evk[j][1]; r over the level's
// extended basis.  With g != 0 the digits are read through the Galois permutation (hoisted
// rotations).  Two adjacent coefficients per lane (16-byte accesses); the permutation keeps
// aligned pairs together (it maps i^1 to src^1).
// `extra` may be the output itself (a running sum): every lane reads its own words before it writes them.
// Where the two words of a_j for positions (i, i + 1) of limb mi come from.  Keys generated with both halves stored
// carry a_j in multiplier form like b_j (word offset a_off inside the key): the kernels read it, one REDC per sum.
// Otherwise it is regenerated from its stream (raw draws, two REDCs per sum).  Both give the same residues.
struct EvkA {
    size_t a_off;     // 0: regenerate
    int kdig;         // digits of a full key: the stream keys start at kdig * nmod * n
};
template <bool SA>
__device__ __forceinline__ ulonglong2 evk_a_words(const u64 *__restrict__ key, const EvkA ea, int nmod, int n, int j, int mi,
                                                  unsigned i, u64 cg0, u64 cg1, u64 bound) {
    ulonglong2 r;
    if (SA) {
        const u64 *ka = key + ea.a_off + ((size_t)j * nmod + mi) * n + i;
        r.x = __builtin_nontemporal_load(ka), r.y = __builtin_nontemporal_load(ka + 1);
    } else {
        const u64 sk_ = key[(size_t)ea.kdig * nmod * n + (size_t)j * nmod + mi];
        r.x = evk_a_draw(sk_, cg0, i, bound), r.y = evk_a_draw(sk_, cg1, i + 1, bound);
    }
    return r;
}
template <bool SA>
__device__ __forceinline__ u64 evk_a_reduce(u128 T, const ModC &m) {
    return SA ? redc(T, m.q, m.qinv) : redc_raw(T, m);
}
static EvkA evk_a_of(const cm_ctx *ctx) {
    return EvkA{ctx->evk_stored_a ? evk_a_offset(ctx) : 0, (ctx->L + ctx->alpha) / ctx->alpha};
}
template <bool SA>
__global__ __launch_bounds__(TPB) void k_inner_product(u64 *u0, u64 *u1,
                                                       const u64 *__restrict__ dig, const u64 *__restrict__ evk,
                                                       const ModC *__restrict__ modc,
                                int beta, int ext, int level, int L, int nmod, int n, int logn, unsigned g,
                                const u64 *__restrict__ c0, const u64 *__restrict__ pmont, const u64 *extra, EvkA eva,
                                const u64 *__restrict__ ubound) {
    unsigned i2 = (blockIdx.x * TPB + threadIdx.x) * 2;
    int r = blockIdx.y;
    int mi = r <= level ? r : L + 1 + (r - level - 1);
    const ModC m = modc[mi];
    unsigned src = g ? perm_src(i2, g, logn) : i2;
    unsigned base = src & ~1u;
    bool swap = src & 1u;
    const u64 bound = ubound[mi], cg0 = ((u64)i2 + 1) * GOLD, cg1 = cg0 + GOLD;
    u128 a0 = 0, a1 = 0, b0 = 0, b1 = 0;
    for (int j = 0; j < beta; j++) {
        ulonglong2 d = *reinterpret_cast<const ulonglong2 *>(dig + ((size_t)j * ext + r) * n + base);
        u64 dx = swap ? d.y : d.x, dy = swap ? d.x : d.y;
        const u64 *kb = evk + ((size_t)j * nmod + mi) * n + i2;
        // the key is streamed once: non-temporal, so that the raised digits (re-read by every
        // hoisted rotation) are the lines that stay in the last-level cache
        ulonglong2 eb;
        eb.x = __builtin_nontemporal_load(kb), eb.y = __builtin_nontemporal_load(kb + 1);
        const ulonglong2 ea = evk_a_words<SA>(evk, eva, nmod, n, j, mi, i2, cg0, cg1, bound);
        b0 += (u128)dx * eb.x;
        b1 += (u128)dy * eb.y;
        a0 += (u128)dx * ea.x;
        a1 += (u128)dy * ea.y;
    }
    if (c0 && r <= level) {           // + P * sigma_g(c0): the rotation stays in the extended basis
        ulonglong2 d = *reinterpret_cast<const ulonglong2 *>(c0 + (size_t)r * n + base);
        const u64 pm = pmont[r];
        b0 += (u128)(swap ? d.y : d.x) * pm;
        b1 += (u128)(swap ? d.x : d.y) * pm;
    }
    size_t o = (size_t)r * n + i2;
    ulonglong2 r0 = make_ulonglong2(redc(b0, m.q, m.qinv), redc(b1, m.q, m.qinv));
    ulonglong2 r1 = make_ulonglong2(evk_a_reduce<SA>(a0, m), evk_a_reduce<SA>(a1, m));
    if (extra) {                      // + a sum already in the extended basis, [2][ext][n]
        ulonglong2 e0 = *reinterpret_cast<const ulonglong2 *>(extra + o);
        ulonglong2 e1 = *reinterpret_cast<const ulonglong2 *>(extra + (size_t)ext * n + o);
        r0.x = addmod(r0.x, e0.x, m.q), r0.y = addmod(r0.y, e0.y, m.q);
        r1.x = addmod(r1.x, e1.x, m.q), r1.y = addmod(r1.y, e1.y, m.q);
    }
    *reinterpret_cast<ulonglong2 *>(u0 + o) = r0;
    *reinterpret_cast<ulonglong2 *>(u1 + o) = r1;
}
// Several inner products in one launch: blockIdx.z = output; output z sums nsum consecutive items
// (each with its own digits, key, Galois element and optional c0) and an optional addend.
// APART (IpBatch::apart) is an instantiation of its own: as a run-time branch it cost all other calls 11 to 15 % of this kernel
// (31 giant steps on 6 limbs of n = 4096, five digits: 51 us without it, 59 with it).
template <bool SA, bool APART>
__global__ __launch_bounds__(TPB) void k_inner_product_batch(IpBatch b, const ModC *__restrict__ modc, int beta, int ext,
                                                             int level, int L, int nmod, int n, int logn,
                                                             const u64 *__restrict__ pmont, EvkA eva,
                                                             const u64 *__restrict__ ubound) {
    // Workgroups go to the eight XCDs round-robin by their linear index.  The rotated reads of the digits gather over
    // a whole limb, and every key of a sum gathers over the same limb again: with a limb's workgroups on ONE XCD (each
    // XCD takes a contiguous eighth of the (limb, block) sequence) those re-reads can hit that XCD's L2.
    unsigned bx = blockIdx.x;
    int r = blockIdx.y;
    if (gridDim.x % 8 == 0) {
        const unsigned lin = blockIdx.x + gridDim.x * blockIdx.y, per = gridDim.x * gridDim.y / 8;
        const unsigned v = (lin & 7u) * per + (lin >> 3);
        bx = v % gridDim.x, r = v / gridDim.x;
    }
    const unsigned i2 = (bx * TPB + threadIdx.x) * 2;
    const int z = blockIdx.z;
    const int mi = r <= level ? r : L + 1 + (r - level - 1);
    const ModC m = modc[mi];
    const size_t o = (size_t)r * n + i2;
    const int special = ext - level - 1, out_rows = APART ? ext + (b.nsum - 1) * special : ext;
    const u64 bound = ubound[mi], cg0 = ((u64)i2 + 1) * GOLD, cg1 = cg0 + GOLD;
    ulonglong2 r0 = make_ulonglong2(0, 0), r1 = make_ulonglong2(0, 0);
    if (!APART && b.extra[z]) {
        r0 = *reinterpret_cast<const ulonglong2 *>(b.extra[z] + o);
        r1 = *reinterpret_cast<const ulonglong2 *>(b.extra[z] + (size_t)ext * n + o);
    }
    for (int s = 0; s < b.nsum; s++) {
        const IpItem it = b.it[z * b.nsum + s];
        const unsigned src = it.g ? perm_src(i2, it.g, logn) : i2;
        const unsigned base = src & ~1u;
        const bool swap = src & 1u;
        u128 a0 = 0, a1 = 0, b0 = 0, b1 = 0;
        for (int j = 0; j < beta; j++) {
            ulonglong2 d = *reinterpret_cast<const ulonglong2 *>(it.dig + ((size_t)j * ext + r) * n + base);
            u64 dx = swap ? d.y : d.x, dy = swap ? d.x : d.y;
            const u64 *kb = it.key + ((size_t)j * nmod + mi) * n + i2;
            ulonglong2 eb;
            eb.x = __builtin_nontemporal_load(kb), eb.y = __builtin_nontemporal_load(kb + 1);
            const ulonglong2 ea = evk_a_words<SA>(it.key, eva, nmod, n, j, mi, i2, cg0, cg1, bound);
            b0 += (u128)dx * eb.x;
            b1 += (u128)dy * eb.y;
            a0 += (u128)dx * ea.x;
            a1 += (u128)dy * ea.y;
        }
        if (it.c0 && it.c0_ext) {            // a first component that never left the extended basis
            ulonglong2 d = *reinterpret_cast<const ulonglong2 *>(it.c0 + (size_t)r * n + base);
            r0.x = addmod(r0.x, swap ? d.y : d.x, m.q), r0.y = addmod(r0.y, swap ? d.x : d.y, m.q);
        } else if (it.c0 && r <= level) {
            ulonglong2 d = *reinterpret_cast<const ulonglong2 *>(it.c0 + (size_t)r * n + base);
            const u64 pm = pmont[r];
            b0 += (u128)(swap ? d.y : d.x) * pm;
            b1 += (u128)(swap ? d.x : d.y) * pm;
        }
        r0.x = addmod(r0.x, redc(b0, m.q, m.qinv), m.q), r0.y = addmod(r0.y, redc(b1, m.q, m.qinv), m.q);
        r1.x = addmod(r1.x, evk_a_reduce<SA>(a0, m), m.q), r1.y = addmod(r1.y, evk_a_reduce<SA>(a1, m), m.q);
        if (APART && r > level) {          // this item's special limb by itself
            u64 *dst = b.out[z] + (size_t)s * special * n + o;
            *reinterpret_cast<ulonglong2 *>(dst) = r0;
            *reinterpret_cast<ulonglong2 *>(dst + (size_t)out_rows * n) = r1;
            r0 = r1 = make_ulonglong2(0, 0);
        }
    }
    if (APART && r > level) return;
    *reinterpret_cast<ulonglong2 *>(b.out[z] + o) = r0;
    *reinterpret_cast<ulonglong2 *>(b.out[z] + (size_t)out_rows * n + o) = r1;
}
// The same key applied to nz digit arrays: a lane keeps its key words in registers and runs over the
// arrays, so the key is read from HBM once per launch.  With g != 0 the digits (and the optional
// it[z].c0, a first component already in the extended basis, added as it is) are read through the
// Galois map; extra[z] ([2][ext][n], may be out[z] itself) is added, which lets several launches with
// different keys accumulate into one output.
#define IP_SHARED_MAX_BETA 8
template <bool SA, int NB>
__global__ __launch_bounds__(TPB) void k_inner_product_shared_key(IpBatch b, const ModC *__restrict__ modc, int beta,
                                                                  int ext, int level, int L, int nmod, int n, int logn,
                                                                  unsigned g, EvkA eva, const u64 *__restrict__ ubound) {
    const unsigned i2 = (blockIdx.x * TPB + threadIdx.x) * 2;
    const int r = blockIdx.y;
    const int mi = r <= level ? r : L + 1 + (r - level - 1);
    const ModC m = modc[mi];
    const size_t o = (size_t)r * n + i2;
    const unsigned src = g ? perm_src(i2, g, logn) : i2;
    const unsigned base = src & ~1u;
    const bool swap = src & 1u;
    ulonglong2 eb[NB], ea[NB];
    const u64 *key = b.it[0].key;
    const u64 bound = ubound[mi], cg0 = ((u64)i2 + 1) * GOLD, cg1 = cg0 + GOLD;
#pragma unroll
    for (int j = 0; j < NB; j++) {
        if (j < beta) {
            const u64 *kb = key + ((size_t)j * nmod + mi) * n + i2;
            eb[j].x = __builtin_nontemporal_load(kb), eb[j].y = __builtin_nontemporal_load(kb + 1);
            ea[j] = evk_a_words<SA>(key, eva, nmod, n, j, mi, i2, cg0, cg1, bound);
        }
    }
    for (int z = 0; z < b.nz; z++) {
        const u64 *dig = b.it[z].dig;
        u128 a0 = 0, a1 = 0, b0 = 0, b1 = 0;
#pragma unroll
        for (int j = 0; j < NB; j++) {
            if (j < beta) {
                ulonglong2 d = *reinterpret_cast<const ulonglong2 *>(dig + ((size_t)j * ext + r) * n + base);
                const u64 dx = swap ? d.y : d.x, dy = swap ? d.x : d.y;
                b0 += (u128)dx * eb[j].x;
                b1 += (u128)dy * eb[j].y;
                a0 += (u128)dx * ea[j].x;
                a1 += (u128)dy * ea[j].y;
            }
        }
        ulonglong2 r0 = make_ulonglong2(redc(b0, m.q, m.qinv), redc(b1, m.q, m.qinv));
        ulonglong2 r1 = make_ulonglong2(evk_a_reduce<SA>(a0, m), evk_a_reduce<SA>(a1, m));
        if (b.it[z].c0) {
            ulonglong2 d = *reinterpret_cast<const ulonglong2 *>(b.it[z].c0 + (size_t)r * n + base);
            r0.x = addmod(r0.x, swap ? d.y : d.x, m.q), r0.y = addmod(r0.y, swap ? d.x : d.y, m.q);
        }
        if (b.extra[z]) {
            ulonglong2 e0 = *reinterpret_cast<const ulonglong2 *>(b.extra[z] + o);
            ulonglong2 e1 = *reinterpret_cast<const ulonglong2 *>(b.extra[z] + (size_t)ext * n + o);
            r0.x = addmod(r0.x, e0.x, m.q), r0.y = addmod(r0.y, e0.y, m.q);
            r1.x = addmod(r1.x, e1.x, m.q), r1.y = addmod(r1.y, e1.y, m.q);
        }
        *reinterpret_cast<ulonglong2 *>(b.out[z] + o) = r0;
        *reinterpret_cast<ulonglong2 *>(b.out[z] + (size_t)ext * n + o) = r1;
    }
}
void launch_inner_product_shared_key(cm_ctx *ctx, const IpBatch &b, int beta, int level, hipStream_t st, u64 g) {
    int ext = level + 1 + ctx->K;
    if (beta > IP_SHARED_MAX_BETA) {          // more digits than a lane keeps: the general batch kernel, one output per array
        IpBatch c = b;
        c.nsum = 1;
        for (int z = 0; z < b.nz; z++) c.it[z].key = b.it[0].key, c.it[z].g = (unsigned)g, c.it[z].c0_ext = c.it[z].c0 ? 1 : 0;
        launch_inner_product_batch(ctx, c, beta, level, st);
        return;
    }
    Prof prof_(ctx, CM_K_INNER_PRODUCT, b.nz, st);
    // NB as in the fan-out kernel: registers for the digits there are
#define SHARED_LAUNCH(SA_, NB_)                                                                                                  \
    hipLaunchKernelGGL((k_inner_product_shared_key<SA_, NB_>), dim3(ctx->n / (2 * TPB), ext), dim3(TPB), 0, st, b, ctx->d_modc, beta, \
                       ext, level, ctx->L, ctx->nmod, ctx->n, ctx->logn, (unsigned)g, evk_a_of(ctx), ctx->d_ubound)
    if (ctx->evk_stored_a) {
        if (beta <= 4) SHARED_LAUNCH(true, 4);
        else SHARED_LAUNCH(true, 8);
    } else if (beta <= 2) SHARED_LAUNCH(false, 2);
    else if (beta <= 3) SHARED_LAUNCH(false, 3);
    else if (beta <= 4) SHARED_LAUNCH(false, 4);
    else if (beta <= 6) SHARED_LAUNCH(false, 6);
    else SHARED_LAUNCH(false, 8);
#undef SHARED_LAUNCH
}
// One digit array, many keys, one output per key (the hoisted rotations of ONE ciphertext, each kept on its own): a lane
// keeps the digit words of two SOURCE positions (and the first component's) in registers and walks over the keys; for
// key a it writes its result at the position the Galois map sends its source to (the inverse map; pairs go to pairs,
// aligned runs of 64 to aligned runs of 64, so key reads and result writes stay coalesced).  Same sums as
// k_inner_product_batch, but the digits are read once per IP_FAN_CHUNK keys instead of once per key.
// NB = compile-time bound of the digit count: registers for eight digits leave three waves a SIMD, each with the two or three
// loads in flight that a low level has; sized for its digits the kernel runs four to eight waves.  Bound by memory (one half
// to two thirds reads): the 63 baby steps of a 4096 x 4096 product at level 4 (two digits) 326 -> 252 us, the 127 of a
// 16384 x 4096 one at level 3 (one digit) 471 -> 362 us.  Requesting the next rotation's words ahead as well changed nothing.
#define IP_FAN_CHUNK 8
template <bool SA, int NB>
__global__ __launch_bounds__(TPB) void k_inner_product_fanout(IpFan f, const u64 *__restrict__ dig, const u64 *__restrict__ c0,
                                                              int c0_ext, const ModC *__restrict__ modc, int beta, int ext,
                                                              int level, int L, int nmod, int n, int logn,
                                                              const u64 *__restrict__ pmont, EvkA eva,
                                                              const u64 *__restrict__ ubound) {
    // The key chunks of one (limb, block) read the same digits: they are given consecutive places in the sequence of
    // ONE XCD (workgroups go to the XCDs round-robin by linear index), so that the digits come from HBM once and from
    // that XCD's L2 for the other chunks.
    unsigned bx = blockIdx.x, bz = blockIdx.z;
    int r = blockIdx.y;
    if (gridDim.x % 8 == 0) {
        const unsigned lin = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z), s = lin >> 3, xs = gridDim.x / 8;
        bz = s % gridDim.z;
        const unsigned rest = s / gridDim.z;
        bx = (lin & 7u) + 8u * (rest % xs), r = rest / xs;
    }
    const unsigned s2 = (bx * TPB + threadIdx.x) * 2;
    const int mi = r <= level ? r : L + 1 + (r - level - 1);
    const ModC m = modc[mi];
    const u64 bound = ubound[mi];
    const bool small = m.q < (1ULL << 50);
    const int a0_ = (int)bz * IP_FAN_CHUNK, a_end = min(f.n, a0_ + IP_FAN_CHUNK);
    struct Words { u64x2 b[NB], a[NB]; };
    ulonglong2 d[NB];
#pragma unroll
    for (int j = 0; j < NB; j++)
        if (j < beta) d[j] = *reinterpret_cast<const ulonglong2 *>(dig + ((size_t)j * ext + r) * n + s2);
    // the first component's contribution to the first output component: sigma(c0) as it is (extended basis) or
    // P sigma(c0) on the ciphertext limbs
    ulonglong2 cv = make_ulonglong2(0, 0);
    const bool have_c0 = c0 && (c0_ext || r <= level);
    if (have_c0) {
        cv = *reinterpret_cast<const ulonglong2 *>(c0 + (size_t)r * n + s2);
        if (!c0_ext) {
            const u64 pm = pmont[r];
            cv.x = redc((u128)cv.x * pm, m.q, m.qinv), cv.y = redc((u128)cv.y * pm, m.q, m.qinv);
        }
    }
    // The generator stream keys of this chunk's (key, digit) pairs: lane 8 a' + j of every wave fetches one, and the loop
    // below broadcasts it with a lane read, so that no draw waits for a load of its own.
    u64 my_sk = 0;
    if (!SA) {
        const int la = (threadIdx.x & 63) >> 3, lj = threadIdx.x & 7;
        static_assert(IP_FAN_CHUNK * IP_SHARED_MAX_BETA == 64, "one lane per (key, digit) of a chunk");
        if (a0_ + la < a_end && lj < beta) my_sk = f.key[a0_ + la][(size_t)eva.kdig * nmod * n + (size_t)lj * nmod + mi];
    }
    for (int a = a0_; a < a_end; a++) {
        const unsigned dst = perm_src(s2, f.ginv[a], logn);       // where this rotation puts source s2; s2 + 1 goes to dst ^ 1
        const unsigned base = dst & ~1u;
        const bool swap = dst & 1u;
        const u64 cg0 = ((u64)base + 1) * GOLD, cg1 = cg0 + GOLD;
        Words w;
        // every key word of this rotation is requested before the first is used
        const u64 *key = f.key[a] + (size_t)mi * n + base;
#pragma unroll
        for (int j = 0; j < NB; j++)
            if (j < beta) {
                const u64 *kb = key + (size_t)j * nmod * n;
                w.b[j] = __builtin_nontemporal_load(reinterpret_cast<const u64x2 *>(kb));
                if (SA) w.a[j] = __builtin_nontemporal_load(reinterpret_cast<const u64x2 *>(kb + eva.a_off));
            }
        if (!SA) {
            // attempt 0 of every draw in straight-line code; the rejected ones (a 2^-14 chance under a 50-bit modulus,
            // up to 1/16 under a 60-bit one) are redone in one branch behind them
            const int l0 = (a - a0_) * 8;
            bool rej = false;
#pragma unroll
            for (int j = 0; j < NB; j++)
                if (j < beta) {
                    const u64 sk_ = ((u64)__builtin_amdgcn_readlane((int)(my_sk >> 32), l0 + j) << 32) |
                                    (unsigned)__builtin_amdgcn_readlane((int)my_sk, l0 + j);
                    w.a[j].x = mix64(sk_ + cg0), w.a[j].y = mix64(sk_ + cg1);
                    rej |= (w.a[j].x >= bound) | (w.a[j].y >= bound);
                }
            if (rej) {
#pragma unroll
                for (int j = 0; j < NB; j++)
                    if (j < beta) {
                        const u64 sk_ = ((u64)__builtin_amdgcn_readlane((int)(my_sk >> 32), l0 + j) << 32) |
                                        (unsigned)__builtin_amdgcn_readlane((int)my_sk, l0 + j);
                        w.a[j].x = evk_a_draw(sk_, cg0, base, bound), w.a[j].y = evk_a_draw(sk_, cg1, base + 1, bound);
                    }
            }
        }
        u128 a0 = 0, a1 = 0, b0 = 0, b1 = 0;
        if (small) {
            Acc50 A0, A1, B0, B1;
#pragma unroll
            for (int j = 0; j < NB; j++) {
                if (j < beta) {
                    const u64 dx = swap ? d[j].y : d[j].x, dy = swap ? d[j].x : d[j].y;      // sources of positions base, base + 1
                    const unsigned x0 = (unsigned)dx & LOW25, x1 = (unsigned)(dx >> 25), y0 = (unsigned)dy & LOW25, y1 = (unsigned)(dy >> 25);
                    B0.mac(x0, x1, w.b[j].x), B1.mac(y0, y1, w.b[j].y);
                    A0.mac(x0, x1, w.a[j].x), A1.mac(y0, y1, w.a[j].y);
                }
            }
            a0 = A0.total(), a1 = A1.total(), b0 = B0.total(), b1 = B1.total();
        } else {
#pragma unroll
            for (int j = 0; j < NB; j++) {
                if (j < beta) {
                    const u64 dx = swap ? d[j].y : d[j].x, dy = swap ? d[j].x : d[j].y;
                    b0 += (u128)dx * w.b[j].x;
                    b1 += (u128)dy * w.b[j].y;
                    a0 += (u128)dx * w.a[j].x;
                    a1 += (u128)dy * w.a[j].y;
                }
            }
        }
        ulonglong2 r0 = make_ulonglong2(redc(b0, m.q, m.qinv), redc(b1, m.q, m.qinv));
        if (have_c0) r0.x = addmod(r0.x, swap ? cv.y : cv.x, m.q), r0.y = addmod(r0.y, swap ? cv.x : cv.y, m.q);
        const size_t o = (size_t)r * n + base;
        // the rotated ciphertexts are read back much later (by the multiply-accumulate kernel): streamed past the caches
        const u64x2 w0 = {r0.x, r0.y}, w1 = {evk_a_reduce<SA>(a0, m), evk_a_reduce<SA>(a1, m)};
        __builtin_nontemporal_store(w0, reinterpret_cast<u64x2 *>(f.out[a] + o));
        __builtin_nontemporal_store(w1, reinterpret_cast<u64x2 *>(f.out[a] + (size_t)ext * n + o));
    }
}
bool launch_inner_product_fanout(cm_ctx *ctx, const IpFan &f, const u64 *dig, const u64 *c0, bool c0_ext, int beta, int level,
                                 hipStream_t st) {
    if (beta > IP_SHARED_MAX_BETA || f.n < 1 || f.n > IP_FAN_MAX) return false;
    Prof prof_(ctx, CM_K_INNER_PRODUCT, f.n, st);
    const int ext = level + 1 + ctx->K;
    const dim3 grid(ctx->n / (2 * TPB), ext, (f.n + IP_FAN_CHUNK - 1) / IP_FAN_CHUNK);
#define FAN_LAUNCH(SA_, NB_)                                                                                                       \
    hipLaunchKernelGGL((k_inner_product_fanout<SA_, NB_>), grid, dim3(TPB), 0, st, f, dig, c0, c0_ext ? 1 : 0, ctx->d_modc, beta, \
                       ext, level, ctx->L, ctx->nmod, ctx->n, ctx->logn, ctx->d_pmont, evk_a_of(ctx), ctx->d_ubound)
    if (ctx->evk_stored_a) {
        if (beta <= 4) FAN_LAUNCH(true, 4);
        else FAN_LAUNCH(true, 8);
    } else if (beta <= 1) FAN_LAUNCH(false, 1);
    else if (beta <= 2) FAN_LAUNCH(false, 2);
    else if (beta <= 3) FAN_LAUNCH(false, 3);
    else if (beta <= 4) FAN_LAUNCH(false, 4);
    else if (beta <= 6) FAN_LAUNCH(false, 6);
    else FAN_LAUNCH(false, 8);
#undef FAN_LAUNCH
    return true;
}
// NA keys (rotation amounts) applied to the same nz digit arrays, summed: out[z] = extra[z] + sum_a [ sum_j
// sigma_a(dig_z,j) key_a,j + (sigma_a(c0_z), 0) ].  A lane keeps the words of all NA keys in registers (at most
// IP_MULTI_BETA digits) and writes every output once: against one launch per amount this saves the read-modify-write
// of the running sum, a third of the traffic of the rotation step of an unrolled ladder.
#define IP_MULTI_BETA 6
template <int NA, bool SA>
__global__ __launch_bounds__(TPB) void k_inner_product_multi_key(IpBatch b, IpKeys ks, const ModC *__restrict__ modc, int beta,
                                                                 int ext, int level, int L, int nmod, int n, int logn, EvkA eva,
                                                                 const u64 *__restrict__ ubound) {
    const unsigned i2 = (blockIdx.x * TPB + threadIdx.x) * 2;
    const int r = blockIdx.y;
    const int mi = r <= level ? r : L + 1 + (r - level - 1);
    const ModC m = modc[mi];
    const size_t o = (size_t)r * n + i2;
    const u64 bound = ubound[mi], cg0 = ((u64)i2 + 1) * GOLD, cg1 = cg0 + GOLD;
    ulonglong2 eb[NA][IP_MULTI_BETA], ea[NA][IP_MULTI_BETA];
    unsigned base[NA];
    bool swap[NA];
#pragma unroll
    for (int a = 0; a < NA; a++) {
        const unsigned src = perm_src(i2, ks.g[a], logn);
        base[a] = src & ~1u, swap[a] = src & 1u;
#pragma unroll
        for (int j = 0; j < IP_MULTI_BETA; j++) {
            if (j < beta) {
                const u64 *kb = ks.key[a] + ((size_t)j * nmod + mi) * n + i2;
                eb[a][j].x = __builtin_nontemporal_load(kb), eb[a][j].y = __builtin_nontemporal_load(kb + 1);
                ea[a][j] = evk_a_words<SA>(ks.key[a], eva, nmod, n, j, mi, i2, cg0, cg1, bound);
            }
        }
    }
    for (int z = 0; z < b.nz; z++) {
        const u64 *dig = b.it[z].dig;
        ulonglong2 r0 = make_ulonglong2(0, 0), r1 = make_ulonglong2(0, 0);
        if (b.extra[z]) {
            r0 = *reinterpret_cast<const ulonglong2 *>(b.extra[z] + o);
            r1 = *reinterpret_cast<const ulonglong2 *>(b.extra[z] + (size_t)ext * n + o);
        }
#pragma unroll
        for (int a = 0; a < NA; a++) {
            u128 a0 = 0, a1 = 0, b0 = 0, b1 = 0;
#pragma unroll
            for (int j = 0; j < IP_MULTI_BETA; j++) {
                if (j < beta) {
                    ulonglong2 d = *reinterpret_cast<const ulonglong2 *>(dig + ((size_t)j * ext + r) * n + base[a]);
                    const u64 dx = swap[a] ? d.y : d.x, dy = swap[a] ? d.x : d.y;
                    b0 += (u128)dx * eb[a][j].x;
                    b1 += (u128)dy * eb[a][j].y;
                    a0 += (u128)dx * ea[a][j].x;
                    a1 += (u128)dy * ea[a][j].y;
                }
            }
            r0.x = addmod(r0.x, redc(b0, m.q, m.qinv), m.q), r0.y = addmod(r0.y, redc(b1, m.q, m.qinv), m.q);
            r1.x = addmod(r1.x, evk_a_reduce<SA>(a0, m), m.q), r1.y = addmod(r1.y, evk_a_reduce<SA>(a1, m), m.q);
            if (b.it[z].c0) {
                ulonglong2 d = *reinterpret_cast<const ulonglong2 *>(b.it[z].c0 + (size_t)r * n + base[a]);
                r0.x = addmod(r0.x, swap[a] ? d.y : d.x, m.q), r0.y = addmod(r0.y, swap[a] ? d.x : d.y, m.q);
            }
        }
        *reinterpret_cast<ulonglong2 *>(b.out[z] + o) = r0;
        *reinterpret_cast<ulonglong2 *>(b.out[z] + (size_t)ext * n + o) = r1;
    }
}
bool launch_inner_product_multi_key(cm_ctx *ctx, const IpBatch &b, const IpKeys &ks, int na, int beta, int level, hipStream_t st) {
    if (beta > IP_MULTI_BETA || na < 2 || na > IP_MULTI_KEYS) return false;
    const int ext = level + 1 + ctx->K;
    const dim3 grid(ctx->n / (2 * TPB), ext), block(TPB);
    Prof prof_(ctx, CM_K_INNER_PRODUCT, b.nz * na, st);
#define MULTI_KEY_LAUNCH(NA_, SA_)                                                                                          \
    hipLaunchKernelGGL((k_inner_product_multi_key<NA_, SA_>), grid, block, 0, st, b, ks, ctx->d_modc, beta, ext, level, ctx->L, \
                       ctx->nmod, ctx->n, ctx->logn, evk_a_of(ctx), ctx->d_ubound)
    if (na == 2 && ctx->evk_stored_a) MULTI_KEY_LAUNCH(2, true);
    else if (na == 2) MULTI_KEY_LAUNCH(2, false);
    else if (ctx->evk_stored_a) MULTI_KEY_LAUNCH(3, true);
    else MULTI_KEY_LAUNCH(3, false);
#undef MULTI_KEY_LAUNCH
    return true;
}
void launch_inner_product_batch(cm_ctx *ctx, const IpBatch &b, int beta, int level, hipStream_t st) {
    Prof prof_(ctx, CM_K_INNER_PRODUCT, b.nz * b.nsum, st);
    int ext = level + 1 + ctx->K;
    const dim3 grid(ctx->n / (2 * TPB), ext, b.nz);
#define BATCH_LAUNCH(SA_, APART_)                                                                                               \
    hipLaunchKernelGGL((k_inner_product_batch<SA_, APART_>), grid, dim3(TPB), 0, st, b, ctx->d_modc, beta, ext, level, ctx->L, ctx->nmod, \
                       ctx->n, ctx->logn, ctx->d_pmont, evk_a_of(ctx), ctx->d_ubound)
    if (ctx->evk_stored_a) {
        if (b.apart) BATCH_LAUNCH(true, true);
        else BATCH_LAUNCH(true, false);
    } else if (b.apart) BATCH_LAUNCH(false, true);
    else BATCH_LAUNCH(false, false);
#undef BATCH_LAUNCH
}
// out[2][ext][n] = (P c0, P c1) on the ciphertext limbs, zero on the special limbs
__global__ void k_raise_by_P(u64 *__restrict__ out, const u64 *__restrict__ in, const ModC *__restrict__ modc,
                             const u64 *__restrict__ pmont, int level, int ext, int n, size_t in_stride, size_t out_stride) {
    int i = blockIdx.x * TPB + threadIdx.x, r = blockIdx.y, c = blockIdx.z & 1;
    in += (blockIdx.z >> 1) * in_stride, out += (blockIdx.z >> 1) * out_stride;      // stacked ciphertexts
    u64 v = 0;
    if (r <= level) {
        const ModC m = modc[r];
        v = redc((u128)in[((size_t)c * (level + 1) + r) * n + i] * pmont[r], m.q, m.qinv);
    }
    out[((size_t)c * ext + r) * n + i] = v;
}
void launch_raise_by_P(cm_ctx *ctx, u64 *out, const u64 *in, int level, hipStream_t st, int count) {
    Prof prof_(ctx, CM_K_ELEMENTWISE, count * 2 * (level + 1 + ctx->K), st);
    int ext = level + 1 + ctx->K;
    hipLaunchKernelGGL(k_raise_by_P, dim3(ctx->n / TPB, ext, 2 * count), dim3(TPB), 0, st, out, in, ctx->d_modc, ctx->d_pmont,
                       level, ext, ctx->n, 2 * (size_t)(level + 1) * ctx->n, 2 * (size_t)ext * ctx->n);
}
void launch_inner_product(cm_ctx *ctx, u64 *u0, u64 *u1, const u64 *dig, const u64 *evk, int beta, int level, u64 g,
                          hipStream_t st, const u64 *c0, const u64 *extra) {
    Prof prof_(ctx, CM_K_INNER_PRODUCT, 1, st);
    int ext = level + 1 + ctx->K;
    if (ctx->evk_stored_a)
        hipLaunchKernelGGL(k_inner_product<true>, dim3(ctx->n / (2 * TPB), ext), dim3(TPB), 0, st, u0, u1, dig, evk, ctx->d_modc,
                           beta, ext, level, ctx->L, ctx->nmod, ctx->n, ctx->logn, (unsigned)g, c0, ctx->d_pmont, extra,
                           evk_a_of(ctx), ctx->d_ubound);
    else
        hipLaunchKernelGGL(k_inner_product<false>, dim3(ctx->n / (2 * TPB), ext), dim3(TPB), 0, st, u0, u1, dig, evk, ctx->d_modc,
                           beta, ext, level, ctx->L, ctx->nmod, ctx->n, ctx->logn, (unsigned)g, c0, ctx->d_pmont, extra,
                           evk_a_of(ctx), ctx->d_ubound);
}

// ---- rescale ---------------------------------------------------------------------------------
// last[comp][n]: coefficient-domain last limb in [0, q_l) -> red[comp][l][n] = last mod q_i
__global__ void k_rescale_reduce(u64 *red, const u64 *last, const ModC *modc, int level, int n) {
    int i = blockIdx.x * TPB + threadIdx.x, l = blockIdx.y, c = blockIdx.z;
    const ModC m = modc[l];
    u64 v = last[(size_t)c * n + i];
    red[((size_t)c * level + l) * n + i] = redc((u128)to_mont(v, m), m.q, m.qinv);
}
// out[comp][l][n] = (in[comp][l] - red[comp][l]) * q_level^{-1}; in has level+1 rows per component
// accumulate: out += the result (out holds a running sum of the same shape)
__global__ void k_rescale_finish(u64 *out, const u64 *in, const u64 *red, const u64 *qlinv, const ModC *modc, int level, int n,
                                 int accumulate) {
    int i = blockIdx.x * TPB + threadIdx.x, l = blockIdx.y, c = blockIdx.z;
    u64 q = modc[l].q;
    u64 d = submod(in[((size_t)c * (level + 1) + l) * n + i], red[((size_t)c * level + l) * n + i], q);
    u64 v = mul_shoup(d, qlinv[2 * l], qlinv[2 * l + 1], q);
    const size_t o = ((size_t)c * level + l) * n + i;
    out[o] = accumulate ? addmod(out[o], v, q) : v;
}
void launch_rescale_reduce(cm_ctx *ctx, u64 *red, const u64 *last, int ncomp, int level, hipStream_t st) {
    Prof prof_(ctx, CM_K_RESCALE, ncomp * level, st);
    hipLaunchKernelGGL(k_rescale_reduce, dim3(ctx->n / TPB, level, ncomp), dim3(TPB), 0, st, red, last, ctx->d_modc, level, ctx->n);
}
void launch_rescale_finish(cm_ctx *ctx, u64 *out, const u64 *in, const u64 *red, const u64 *d_qlinv, int ncomp, int level, hipStream_t st,
                           bool accumulate) {
    Prof prof_(ctx, CM_K_RESCALE, ncomp * level, st);
    hipLaunchKernelGGL(k_rescale_finish, dim3(ctx->n / TPB, level, ncomp), dim3(TPB), 0, st, out, in, red, d_qlinv, ctx->d_modc, level, ctx->n,
                       accumulate ? 1 : 0);
}

// ---- counter-based sampling (must reproduce the generator's published definition bit for bit) --------
u64 rng_key(u64 seed, u64 stream) { return mix64(mix64(seed) ^ stream); }
u64 rng_draw(u64 key, u64 ctr) { return mix64(key + (ctr + 1) * GOLD); }

// uniform residues: row l uses stream stream_base | mod_idx[l]
__global__ void k_sample_uniform(u64 *out, const int *mod_idx, const ModC *modc, int n, u64 mseed, u64 stream_base) {
    int i = blockIdx.x * TPB + threadIdx.x, l = blockIdx.y;
    int mi = mod_idx[l];
    u64 q = modc[mi].q;
    u64 key = mix64(mseed ^ (stream_base | (u64)mi));
    // bound = q * floor(2^64 / q): floor(2^64/q) = floor((2^64 - 1)/q) because q is odd > 1
    u64 bound = q * (0xFFFFFFFFFFFFFFFFULL / q);
    u64 att = 0, v;
    do {
        v = mix64(key + (((att << 32) | (u64)i) + 1) * GOLD);
        att++;
    } while (v >= bound);
    out[(size_t)l * n + i] = v % q;
}
void launch_sample_uniform(cm_ctx *ctx, u64 *out, const int *d_mod_idx, int limbs, u64 seed, u64 stream_base, hipStream_t st) {
    hipLaunchKernelGGL(k_sample_uniform, dim3(ctx->n / TPB, limbs), dim3(TPB), 0, st, out, d_mod_idx, ctx->d_modc, ctx->n,
                       mix64(seed), stream_base);
}
// one Gaussian integer per coefficient, written as residues to every row
__global__ void k_sample_gauss(u64 *out, const int *mod_idx, const ModC *modc, const u64 *cdt, int limbs, int n, u64 key) {
    int i = blockIdx.x * TPB + threadIdx.x;
    u64 v = mix64(key + ((u64)i + 1) * GOLD), u = v >> 1;
    u64 mag = 0;
    for (int k = 0; k < CM_GAUSS_K; k++) mag += (u >= cdt[k]);
    bool neg = (v & 1) && mag;
    for (int l = 0; l < limbs; l++) {
        u64 q = modc[mod_idx[l]].q;
        out[(size_t)l * n + i] = neg ? q - mag : mag;
    }
}
void launch_sample_gauss(cm_ctx *ctx, u64 *out, const int *d_mod_idx, int limbs, u64 seed, u64 stream, hipStream_t st) {
    hipLaunchKernelGGL(k_sample_gauss, dim3(ctx->n / TPB), dim3(TPB), 0, st, out, d_mod_idx, ctx->d_modc, ctx->d_cdt, limbs,
                       ctx->n, rng_key(seed, stream));
}

// ---- keys and encryption ---------------------------------------------------------------------------
// b = e - a s + fac_l * s_from, then (b, a) stored in multiplier form.  s_mont: secret, evaluation
// domain, multiplier form, rows = all moduli.  s_from = s through the Galois map g (g != 0) or s^2.
__global__ void k_evk_assemble(u64 *b_out, const u64 *a_in, const u64 *e, const u64 *s_mont, const u64 *fac,
                               const ModC *modc, int n, int logn, unsigned g) {
    unsigned i = blockIdx.x * TPB + threadIdx.x;
    int l = blockIdx.y;
    const ModC m = modc[l];
    size_t o = (size_t)l * n + i;
    u64 a = a_in[o];
    u64 b = submod(e[o], redc((u128)a * s_mont[o], m.q, m.qinv), m.q);
    u64 f = fac[l];
    if (f) {
        u64 sf = g ? s_mont[(size_t)l * n + perm_src(i, g, logn)]
                   : redc((u128)s_mont[o] * s_mont[o], m.q, m.qinv);      // s^2 in multiplier form
        b = addmod(b, redc((u128)f * sf, m.q, m.qinv), m.q);
    }
    b_out[o] = to_mont(b, m);
}
void launch_evk_assemble(cm_ctx *ctx, u64 *b_out, const u64 *a_in, const u64 *e, const u64 *s_mont, const u64 *d_fac, u64 g, hipStream_t st) {
    hipLaunchKernelGGL(k_evk_assemble, dim3(ctx->n / TPB, ctx->nmod), dim3(TPB), 0, st, b_out, a_in, e, s_mont, d_fac,
                       ctx->d_modc, ctx->n, ctx->logn, (unsigned)g);
}
// c0 = e - a s + m
__global__ void k_encrypt(u64 *c0, const u64 *a, const u64 *e, const u64 *s_mont, const u64 *pt, const ModC *modc, int n) {
    int i = blockIdx.x * TPB + threadIdx.x, l = blockIdx.y;
    const ModC m = modc[l];
    size_t o = (size_t)l * n + i;
    u64 v = submod(e[o], redc((u128)a[o] * s_mont[o], m.q, m.qinv), m.q);
    c0[o] = addmod(v, pt[o], m.q);
}
void launch_encrypt(cm_ctx *ctx, u64 *c0, const u64 *a, const u64 *e, const u64 *s_mont, const u64 *pt, int limbs, hipStream_t st) {
    hipLaunchKernelGGL(k_encrypt, dim3(ctx->n / TPB, limbs), dim3(TPB), 0, st, c0, a, e, s_mont, pt, ctx->d_modc, ctx->n);
}
// out = c0 + c1 s (+ c2 s^2) on the first `limbs` limbs; ct rows per component = ct_limbs
__global__ void k_decrypt(u64 *out, const u64 *ct, const u64 *s_mont, const ModC *modc, int ncomp, int ct_limbs, int n) {
    int i = blockIdx.x * TPB + threadIdx.x, l = blockIdx.y;
    const ModC m = modc[l];
    size_t o = (size_t)l * n + i, cs = (size_t)ct_limbs * n;
    u64 s = s_mont[o];
    u64 acc = addmod(ct[o], redc((u128)ct[o + cs] * s, m.q, m.qinv), m.q);
    if (ncomp == 3) {
        u64 s2 = redc((u128)s * s, m.q, m.qinv);
        acc = addmod(acc, redc((u128)ct[o + 2 * cs] * s2, m.q, m.qinv), m.q);
    }
    out[o] = acc;
}
void launch_decrypt(cm_ctx *ctx, u64 *out, const u64 *ct, const u64 *s_mont, int ncomp, int ct_limbs, int limbs, hipStream_t st) {
    hipLaunchKernelGGL(k_decrypt, dim3(ctx->n / TPB, limbs), dim3(TPB), 0, st, out, ct, s_mont, ctx->d_modc, ncomp, ct_limbs, ctx->n);
}

// ---- packed product: inner_k = sum_j baby_j * p_{j,k} ---------------------------------------------------
// babies: r_i ciphertexts [2][limbs][n] at stride ct_stride; out: r_o ciphertexts at stride
// ct_stride; pts: the r_i*r_o plaintexts in multiplier form, blocked for streaming:
//     the words of plaintexts (8g .. 8g+7, k) of chunk ch (64 coefficients) of limb l are one group, the groups follow each
// other in k, g, ch, l: a wave that takes some k of one g, and the workgroup that owns (l, ch), read contiguous stretches.
// Limb l has modulus index l up to `level`, and the special primes follow when limbs = level + 1 + K (sums
// kept in the extended basis).
#define MAC_CO 64
#define MAC_G 8       // plaintexts of a group: what a lane loads at once for one giant step
// Bound by HBM, and by what writes do to a read stream there: plain kernels read 7.1 TB/s with non-temporal loads (6.4 without
// them), but 5 GB read with 3 % of stores sprinkled over the launch take 924 us instead of 744, whatever the stores' size or
// placement; 881 if the stores go through to memory at once (agent scope) instead of leaving the L2 when it evicts them.
// Arithmetic, LDS reads and barriers are hidden: without them, the plaintext stream and the stores alone take as long.
// So bytes count: the packed groups, and the stores at agent scope.  Per launch, before (FP64 products on the limbs below
// 2^50, 128-bit sums and 64-bit words on the others, plain stores) -> now: 64 x 8 products at level 23 1597 -> 1419 us, at
// level 4 540 -> 471, 128 x 16 at level 3 1644 -> 1365, 64 x 16 (32 tokens of 1024 x 1024) at level 9 1438 -> 1278.
// Sums of a wave that keeps all baby words of a group in registers (no LDS, no barriers), two or three groups in flight, FP64
// or integer: within 2 % of this or slower.
// Where there are at least eight baby steps the groups of limbs below 2^60 are packed, so that all loads are aligned and cover
// whole lines a wave:
//   below 2^50: eight words of a coefficient as their low 32 bits (two 16-byte lane words, 1 KiB a wave each), the next 16
//               bits (one) and the top two bits (one halfword), 50 bytes instead of 64;
//   below 2^60: the sixteen 30-bit halves in fifteen 32-bit words (three 16-byte lane words and one of 12), the last half in
//               the top two bits of each, 60 bytes.
// Fewer baby steps and larger moduli keep 64-bit words: with an even number of baby steps, the words of plaintexts (2j', k) and
// (2j'+1, k) are interleaved (word c of the pair at 2c, 2c+1 of a 128-word row), so that a lane reads both with one 16-byte load.
#define MAC_PACK50_WORDS 400                   // 64-bit words of a packed group: 64 coefficients x 8 plaintexts
#define MAC_PACK60_WORDS 480
struct MacLayout {
    int n, r_i, r_o;
    u64 packed50, packed60;                    // bit l: how limb l is packed
    __host__ __device__ __forceinline__ bool is50(int l) const { return (packed50 >> l) & 1; }
    __host__ __device__ __forceinline__ bool is60(int l) const { return (packed60 >> l) & 1; }
    __host__ __device__ __forceinline__ int per_group() const { return r_i % MAC_G ? r_i : MAC_G; }     // plaintexts of a group
    __host__ __device__ __forceinline__ int group_words(int l) const {
        return is50(l) ? MAC_PACK50_WORDS : is60(l) ? MAC_PACK60_WORDS : per_group() * MAC_CO;
    }
    __host__ __device__ __forceinline__ size_t groups() const { return (size_t)(n / MAC_CO) * r_o * (r_i / per_group()); }     // of a limb
    __host__ __device__ __forceinline__ size_t limb_words(int l) const { return groups() * group_words(l); }
    // first word of group g (baby steps 8 g ..) of giant step k of chunk ch of limb l
    __host__ __device__ __forceinline__ size_t group(int l, int ch, int g, int k) const {
        const u64 below = (1ULL << l) - 1;
        const int b50 = __builtin_popcountll(packed50 & below), b60 = __builtin_popcountll(packed60 & below);
        return groups() * ((size_t)b50 * MAC_PACK50_WORDS + (size_t)b60 * MAC_PACK60_WORDS + (size_t)(l - b50 - b60) * per_group() * MAC_CO) +
               (((size_t)ch * (r_i / per_group()) + g) * r_o + k) * group_words(l);
    }
    // unpacked limbs: word (j, c) of a group
    __host__ __device__ __forceinline__ int word(int j, int c) const {
        return (r_i & 1) ? j * MAC_CO + c : (j & ~1) * MAC_CO + 2 * c + (j & 1);
    }
};
static MacLayout mac_layout(const cm_ctx *ctx, int r_i, int r_o, int limbs, int level) {
    MacLayout m{ctx->n, r_i, r_o, 0, 0};
    if (r_i % MAC_G == 0)
        for (int l = 0; l < limbs; l++) {
            const u64 q = ctx->mod[l <= level ? l : ctx->L + (l - level)];
            if (q < (1ULL << 50)) m.packed50 |= 1ULL << l;
            else if (q < (1ULL << 60)) m.packed60 |= 1ULL << l;
        }
    return m;
}
size_t vmm_pts_words(const cm_ctx *ctx, int r_i, int r_o, int limbs, int level) {
    const MacLayout m = mac_layout(ctx, r_i, r_o, limbs, level);
    size_t w = 0;
    for (int l = 0; l < limbs; l++) w += m.limb_words(l);
    return w;
}
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
// Both factors of a product are split, so that it is four 32 x 32 -> 64-bit multiply-adds into three accumulators without
// carries: T = t0 + 2^B t1 + 2^2B t2 with B = 25 under the 50-bit primes, 30 under the others.
struct MacAcc {
    u64 t0 = 0, t1 = 0, t2 = 0;
    __device__ __forceinline__ void mac(unsigned b0, unsigned b1, unsigned w0, unsigned w1) {
        t0 += (u64)b0 * w0, t1 += (u64)b0 * w1, t1 += (u64)b1 * w0, t2 += (u64)b1 * w1;
    }
    template <int B>
    __device__ __forceinline__ u64 reduce(const ModC &m) const {
        return redc((u128)t0 + ((u128)t1 << B) + ((u128)t2 << (2 * B)), m.q, m.qinv);
    }
};
// A lane's eight words of a group; B: bits of the lower half; TERMS: products that the accumulators hold (t1 takes two a term).
struct MacPacked50 {
    static constexpr int GROUP_WORDS = MAC_PACK50_WORDS, B = 25, TERMS = 1 << 13;
    u32x4 lo0, lo1, mid;
    unsigned top;
    __device__ __forceinline__ void load(const u64 *grp, int co) {
        const u32x4 *v = reinterpret_cast<const u32x4 *>(grp);
        lo0 = __builtin_nontemporal_load(v + co), lo1 = __builtin_nontemporal_load(v + 64 + co);
        mid = __builtin_nontemporal_load(v + 128 + co);
        top = __builtin_nontemporal_load(reinterpret_cast<const unsigned short *>(v + 192) + co);
    }
    __device__ __forceinline__ void word(int j, unsigned &w0, unsigned &w1) const {
        const unsigned lo = j < 4 ? lo0[j & 3] : lo1[j & 3], m = mid[j >> 1];
        const unsigned hi = (((top >> (2 * j)) & 3u) << 16) | ((j & 1) ? m >> 16 : m & 0xFFFFu);
        w0 = lo & LOW25, w1 = __builtin_amdgcn_alignbit(hi, lo, 25);
    }
};
typedef unsigned u32x3 __attribute__((ext_vector_type(3), aligned(4)));
struct MacPacked60 {
    static constexpr int GROUP_WORDS = MAC_PACK60_WORDS, B = 30, TERMS = 8;
    u32x4 a[3];
    u32x3 b;
    unsigned last;
    __device__ __forceinline__ void load(const u64 *grp, int co) {
        const u32x4 *v = reinterpret_cast<const u32x4 *>(grp);
#pragma unroll
        for (int i = 0; i < 3; i++) a[i] = __builtin_nontemporal_load(v + 64 * i + co);
        b = __builtin_nontemporal_load(reinterpret_cast<const u32x3 *>((const char *)grp + 3072 + 12 * co));
    }
    __device__ __forceinline__ unsigned d(int i) const { return i < 12 ? a[i / 4][i % 4] : b[i % 4]; }
    __device__ __forceinline__ void word(int j, unsigned &w0, unsigned &w1) const {
        w0 = d(2 * j) & LOW30;
        if (j < 7) {
            w1 = d(2 * j + 1) & LOW30;
        } else {
            w1 = 0;
#pragma unroll
            for (int i = 0; i < 15; i++) w1 = __builtin_amdgcn_alignbit(w1, d(i), 30);
        }
    }
};
struct MacWords {                              // 64-bit words, pairs interleaved: moduli from 2^60 up to 2^61
    static constexpr int GROUP_WORDS = MAC_G * MAC_CO, B = 30, TERMS = 4;
    u64x2 w[MAC_G / 2];
    __device__ __forceinline__ void load(const u64 *grp, int co) {
#pragma unroll
        for (int i = 0; i < MAC_G / 2; i++) w[i] = __builtin_nontemporal_load(reinterpret_cast<const u64x2 *>(grp) + 64 * i + co);
    }
    __device__ __forceinline__ void word(int j, unsigned &w0, unsigned &w1) const {
        const u64 v = (j & 1) ? w[j / 2].y : w[j / 2].x;
        w0 = (unsigned)v & LOW30, w1 = (unsigned)(v >> 30);
    }
};
// An item is 64 coefficients of one limb and W * KW giant steps, KW to each of a workgroup's W waves.  The baby words are staged in LDS
// as two halves, sixteen baby steps a pass (16 KiB), the first group of a pass requested before them.  The sums stay in registers over
// the passes and go to put(giant step, component, sum).
#define MAC_JC 16
template <int W, int KW, class G, class PUT>
__device__ __forceinline__ void mac_body(uint2 *sb, const u64 *__restrict__ babies, const u64 *__restrict__ pts, const ModC &m,
                                         const MacLayout &lay, int l, int ch, int kb, bool first, size_t cs, size_t ct_stride, PUT put) {
    const int co = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const size_t o = (size_t)l * lay.n + ch * MAC_CO;          // uniform: lanes differ by co alone
    const bool active = kb < lay.r_o;                         // uniform in a wave
    u64 s[KW][2];
#pragma unroll
    for (int k = 0; k < KW; k++) s[k][0] = s[k][1] = 0;
    for (int j0 = 0; j0 < lay.r_i; j0 += MAC_JC) {
        const int groups = min(MAC_JC, lay.r_i - j0) / MAC_G, rows = 2 * MAC_G * groups;
        const u64 *p = pts + lay.group(l, ch, j0 / MAC_G, kb);
        G q;
        if (active) q.load(p, co);                            // in flight across the staging
        {
            // a lane stages word `co` of rows wave, wave + W, ...: all its loads are issued before the first is used
            constexpr int ROWS = MAC_JC * 2 / W;
            u64 x[ROWS];
#pragma unroll
            for (int it = 0; it < ROWS; it++) {
                const int r = min(wave + W * it, rows - 1);                 // past the last row: one more time, never used
                x[it] = __builtin_nontemporal_load(babies + (size_t)(j0 + (r >> 1)) * ct_stride + (r & 1) * cs + o + co);
            }
            if (j0 || !first) __syncthreads();
#pragma unroll
            for (int it = 0; it < ROWS; it++)
                sb[(wave + W * it) * MAC_CO + co] = make_uint2((unsigned)x[it] & ((1u << G::B) - 1), (unsigned)(x[it] >> G::B));
            __syncthreads();
        }
        if (!active) continue;
#pragma unroll
        for (int k = 0; k < KW; k++) {
            MacAcc t[2];
#pragma unroll 1
            for (int g = 0; g < groups; g++) {
                G nx = q;
                // the next group is in flight while this one is multiplied
                if (g + 1 < groups) nx.load(p + ((size_t)(g + 1) * lay.r_o + k) * G::GROUP_WORDS, co);
                else if (k + 1 < KW) nx.load(p + (size_t)(k + 1) * G::GROUP_WORDS, co);
#pragma unroll
                for (int j = 0; j < MAC_G; j++) {
                    unsigned w0, w1;
                    q.word(j, w0, w1);
#pragma unroll
                    for (int c = 0; c < 2; c++) {
                        const uint2 b = sb[((g * MAC_G + j) * 2 + c) * MAC_CO + co];
                        t[c].mac(b.x, b.y, w0, w1);
                    }
                    if (G::TERMS <= MAC_G && (j + 1) % G::TERMS == 0) {
#pragma unroll
                        for (int c = 0; c < 2; c++) s[k][c] = addmod(s[k][c], t[c].template reduce<G::B>(m), m.q), t[c] = MacAcc();
                    }
                }
                q = nx;
            }
            if (G::TERMS > MAC_G) {
#pragma unroll
                for (int c = 0; c < 2; c++) s[k][c] = addmod(s[k][c], t[c].template reduce<G::B>(m), m.q);
            }
        }
    }
    if (!active) return;
#pragma unroll
    for (int k = 0; k < KW; k++) put(k, 0, s[k][0]), put(k, 1, s[k][1]);
}
__device__ __forceinline__ void mac_store(u64 *p, u64 v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// A workgroup for every 64 coefficients of a limb, which runs over the blocks of W * KW giant steps and writes as it goes.
template <int W, int KW>
__global__ __launch_bounds__(64 * W) void k_vmm_mac_direct(u64 *__restrict__ out, const u64 *__restrict__ babies, const u64 *__restrict__ pts,
                                                           const ModC *__restrict__ modc, MacLayout lay, int limbs, size_t ct_stride, int level, int L) {
    __shared__ uint2 sb[MAC_JC * 2 * MAC_CO];
    // the limbs of the special primes (60 or 64 bits a word, the slowest workgroups) are dispatched first, not last
    const int nsp = limbs - (level + 1), y = blockIdx.y, ch = blockIdx.x;
    const int l = y < nsp ? level + 1 + y : y - nsp;
    const ModC m = modc[l <= level ? l : L + 1 + (l - level - 1)];
    const size_t cs = (size_t)limbs * lay.n, o = (size_t)l * lay.n + ch * MAC_CO;          // uniform: lanes differ by their coefficient alone
    auto run = [&](auto g) {
        for (int k0 = 0; k0 < lay.r_o; k0 += W * KW) {
            const int kb = k0 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * KW;
            auto put = [=](int k, int c, u64 v) { mac_store(out + (size_t)(kb + k) * ct_stride + c * cs + o + (threadIdx.x & 63), v); };
            mac_body<W, KW, decltype(g)>(sb, babies, pts, m, lay, l, ch, kb, k0 == 0, cs, ct_stride, put);
        }
    };
    if (lay.is50(l)) run(MacPacked50());
    else if (lay.is60(l)) run(MacPacked60());
    else run(MacWords());
}
// Bound by HBM, whose reads the writes disturb: 3 % of the bytes written while others read cost 20 % of a launch, the same bytes written
// when nobody reads cost little (a plain kernel that reads 5 GB and writes 5 %: 789 us without its writes, 1012 with them spread over
// the launch, 844 and 857 as four and eight launches that write last).  So a launch is what the chip holds at once (16 waves a compute
// unit: 108 and 124 registers), `wgs` workgroups of `rounds` <= P items each, P by the LDS (40 KiB and 64 KiB a workgroup), and all
// of them write at its end.  Against k_vmm_mac_direct: 512 products at levels 23 and 4 1413 -> 1300 and 470 -> 431 us, 2048 at level 3
// 1359 -> 1305, 1024 at level 9 1267 -> 1155, three times 128 at level 13 292 -> 268 each (vmm_mac_held: where not); one launch that writes
// after every third item 1439, 448, 1344, 1208 and 282.  P = 8 with eight waves for eight giant steps, P = 4 for sixteen: within 2 %.
// Item `round` of a workgroup: chunk and limb by unit, then the block of W * KW giant steps.
struct MacArgs {
    int wgs, round, rounds, blocks;
};
template <int W, int KW, int P>
__global__ __launch_bounds__(64 * W, 4) void k_vmm_mac(u64 *__restrict__ out, const u64 *__restrict__ babies, const u64 *__restrict__ pts,
                                                       const ModC *__restrict__ modc, MacLayout lay, MacArgs a, int limbs, size_t ct_stride,
                                                       int level, int L) {
    __shared__ uint2 sb[MAC_JC * 2 * MAC_CO];
    __shared__ u64 res[P * W * KW * 2 * MAC_CO];
    const int chunks = lay.n / MAC_CO, nsp = limbs - (level + 1);
    const int co = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const size_t cs = (size_t)limbs * lay.n;
    // the limbs of the special primes (60 or 64 bits a word) come first
    auto item = [&](int i, int &l, int &ch, int &kb) {
        const int r = a.round + i, u = (int)blockIdx.x + a.wgs * (r / a.blocks), y = u / chunks;
        l = y < nsp ? level + 1 + y : y - nsp, ch = u % chunks, kb = ((r % a.blocks) * W + wave) * KW;
        return y < limbs;
    };
    for (int i = 0; i < a.rounds; i++) {
        int l, ch, kb;
        if (!item(i, l, ch, kb)) break;
        const ModC m = modc[l <= level ? l : L + 1 + (l - level - 1)];
        u64 *r = res + ((i * W + wave) * KW * 2) * MAC_CO + co;
        auto put = [&](int k, int c, u64 v) { r[(2 * k + c) * MAC_CO] = v; };             // a lane reads back what it wrote
        if (lay.is50(l)) mac_body<W, KW, MacPacked50>(sb, babies, pts, m, lay, l, ch, kb, i == 0, cs, ct_stride, put);
        else if (lay.is60(l)) mac_body<W, KW, MacPacked60>(sb, babies, pts, m, lay, l, ch, kb, i == 0, cs, ct_stride, put);
        else mac_body<W, KW, MacWords>(sb, babies, pts, m, lay, l, ch, kb, i == 0, cs, ct_stride, put);
    }
    for (int i = 0; i < a.rounds; i++) {
        int l, ch, kb;
        if (!item(i, l, ch, kb)) break;
        if (kb >= lay.r_o) continue;
        const u64 *r = res + ((i * W + wave) * KW * 2) * MAC_CO + co;
        const size_t o = (size_t)l * lay.n + ch * MAC_CO + co;
#pragma unroll
        for (int k = 0; k < KW; k++)
#pragma unroll
            for (int c = 0; c < 2; c++) mac_store(out + (size_t)(kb + k) * ct_stride + c * cs + o, r[(2 * k + c) * MAC_CO]);
    }
}
// Fewer than eight baby steps (RI = 1, 2 or 4): a lane keeps its baby words and runs over MAC_FEW_K giant steps, the words of the
// next one requested ahead.  Bound by HBM, mostly by the sums it writes (2 words for RI read), so these are stored at agent scope.
// 512 products at level 4, RI = 1, 2, 4 (2.7, 1.3 and 0.7 GB written, 1.3 GB read): 737, 477 and 353 us; with 8-byte loads at stride two
// and plain stores 752, 692 and 564; in the kernel for eight baby steps and more (with 128-bit sums) 1141, 554 and 371.  32 x 4 at n = 4096:
// 14 us, 24, 20.  Four giant steps a lane: 4 % slower to 4 % faster; sixteen: 2 % faster, and 30 % slower at n = 4096.
#define MAC_FEW_K 8
template <int RI>
__global__ __launch_bounds__(TPB) void k_vmm_mac_few(u64 *__restrict__ out, const u64 *__restrict__ babies, const u64 *__restrict__ pts,
                                                    const ModC *__restrict__ modc, MacLayout lay, int limbs, size_t ct_stride, int level,
                                                    int L) {
    const int l = blockIdx.y, i = blockIdx.x * TPB + threadIdx.x, mi = l <= level ? l : L + 1 + (l - level - 1);
    const ModC m = modc[mi];
    const size_t o = (size_t)l * lay.n + i, cs = (size_t)limbs * lay.n;
    const int k0 = blockIdx.z * MAC_FEW_K, k1 = min(k0 + MAC_FEW_K, lay.r_o);
    const u64 *run = pts + lay.group(l, i / MAC_CO, 0, k0);              // the groups of a chunk's giant steps follow each other
    auto load = [&](int k, u64 (&w)[RI]) {
        const u64 *p = run + (size_t)(k - k0) * (RI * MAC_CO);
        if (RI == 1) w[0] = __builtin_nontemporal_load(p + i % MAC_CO);
#pragma unroll
        for (int j = 0; j + 1 < RI; j += 2) {
            const u64x2 v = __builtin_nontemporal_load(reinterpret_cast<const u64x2 *>(p + j * MAC_CO) + i % MAC_CO);
            w[j] = v.x, w[j + 1] = v.y;
        }
    };
    u64 b[RI][2], w[RI], nx[RI];
    load(k0, w);
#pragma unroll
    for (int j = 0; j < RI; j++)
#pragma unroll
        for (int c = 0; c < 2; c++) b[j][c] = babies[j * ct_stride + c * cs + o];
    for (int k = k0; k < k1; k++) {
        if (k + 1 < k1) load(k + 1, nx);
        u128 s0 = 0, s1 = 0;                   // four products: below q 2^64 for all moduli
#pragma unroll
        for (int j = 0; j < RI; j++) s0 += (u128)b[j][0] * w[j], s1 += (u128)b[j][1] * w[j], w[j] = nx[j];
        __hip_atomic_store(out + k * ct_stride + o, redc(s0, m.q, m.qinv), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(out + k * ct_stride + cs + o, redc(s1, m.q, m.qinv), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}
// Held sums gain where the plaintexts outweigh what is written, 2 words of sums to r_i of plaintext a giant step, and lose where the chip waits
// for the last item of every launch.  Held against direct, us, (limbs, r_i, r_o) at n = 65536: (28, 32, 16) 1190, 1365; (9, 32, 16) 397,
// 420; (9, 64, 2) 183, 192; (3, 32, 2) 32.3, 32.0; one giant step (9, 64, 1) 147, 142; (28, 8, 1) 127, 82; (28, 8, 32) 917, 813; sixteen
// baby steps (9, 16, 8) 122, 127; (28, 16, 4) 228, 228; (9, 16, 2) 55.7, 52.1; (6, 16, 8) 84.6, 83.7; (6, 16, 64) 640, 691; (14, 16, 16)
// 326, 321; (18, 16, 16) 441, 468.  Two, four and eight limbs put the ciphertexts of a sum at distances of a power of two, which a
// resident set that works on one limb feels: (8, 32, 4) 128.8, 126.6; (4, 16, 8) 56.8, 51.6; (8, 64, 8) 382, 395.  At n = 4096 (14, 32, 64) 154,
// 159; (7, 16, 16) 13.3, 12.5; (4, 64, 8) 21.4, 20.1.
bool vmm_mac_held(int n, int limbs, int r_i, int r_o) {
    if (n == 4096) return r_i >= 32 && r_o >= 32 && limbs >= 14;
    if (r_i < 16 || r_o < 2) return false;
    const bool pow2 = !(limbs & (limbs - 1)) && limbs <= 8;
    if (r_i > 16) return !pow2 || r_i * r_o >= 512;
    return r_o >= 64 ? limbs >= 5 : r_o == 16 ? limbs > 16 : r_o >= 4 && limbs >= 7 && !pow2;
}
void launch_vmm_mac(cm_ctx *ctx, u64 *out, const u64 *babies, const u64 *pts, int r_i, int r_o, int limbs, int level,
                    size_t ct_stride, hipStream_t st) {
    launch_vmm_mac_form(ctx, out, babies, pts, r_i, r_o, limbs, level, ct_stride, st, vmm_mac_held(ctx->n, limbs, r_i, r_o));
}
void launch_vmm_mac_form(cm_ctx *ctx, u64 *out, const u64 *babies, const u64 *pts, int r_i, int r_o, int limbs, int level,
                         size_t ct_stride, hipStream_t st, bool held) {
    Prof prof_(ctx, CM_K_VMM_MAC, r_i * r_o, st);
    const MacLayout lay = mac_layout(ctx, r_i, r_o, limbs, level);
    if (r_i % 8) {
        const dim3 few(ctx->n / TPB, limbs, (r_o + MAC_FEW_K - 1) / MAC_FEW_K);
#define FEW_LAUNCH(RI_) hipLaunchKernelGGL(k_vmm_mac_few<RI_>, few, dim3(TPB), 0, st, out, babies, pts, ctx->d_modc, lay, limbs, ct_stride, level, ctx->L)
        if (r_i == 1) FEW_LAUNCH(1);
        else if (r_i == 2) FEW_LAUNCH(2);
        else FEW_LAUNCH(4);
#undef FEW_LAUNCH
        return;
    }
    if (!held) {
        const dim3 grid(ctx->n / MAC_CO, limbs);
#define DIRECT_LAUNCH(W_, KW_) hipLaunchKernelGGL((k_vmm_mac_direct<W_, KW_>), grid, dim3(64 * W_), 0, st, out, babies, pts, ctx->d_modc, lay, limbs, ct_stride, level, ctx->L)
        // n = 4096 leaves compute units idle, which eight waves of half the giant steps use: (limbs, r_i, r_o) (2, 32, 16) 14.4 -> 10.9 us,
        // (4, 16, 32) 18.4 -> 15.2, (26, 32, 64) 314 -> 302; not (5, 8, 16) 7.5 -> 8.0 and (14, 8, 16) 14.3 -> 15.1, nor n = 65536 (5, 8, 16) 64.8 -> 69.0
        if (r_o <= 4) DIRECT_LAUNCH(4, 1);
        else if (r_o <= 8) DIRECT_LAUNCH(4, 2);
        else if (ctx->n == 4096 && (r_i >= 16 || r_o > 16 || limbs <= 4)) DIRECT_LAUNCH(8, 2);
        else DIRECT_LAUNCH(4, 4);
#undef DIRECT_LAUNCH
        return;
    }
    auto launch = [&](auto kernel, int waves, int per, int hold) {
        const int units = ctx->n / MAC_CO * limbs, wgs = std::min(units, 256 * 16 / waves), blocks = (r_o + per - 1) / per;
        const int rounds = (units + wgs - 1) / wgs * blocks, launches = (rounds + hold - 1) / hold;
        for (int i = 0; i < launches; i++) {
            const int r0 = (int)((long long)rounds * i / launches), r1 = (int)((long long)rounds * (i + 1) / launches);
            hipLaunchKernelGGL(kernel, dim3(wgs), dim3(64 * waves), 0, st, out, babies, pts, ctx->d_modc, lay, MacArgs{wgs, r0, r1 - r0, blocks},
                               limbs, ct_stride, level, ctx->L);
        }
    };
    if (r_o <= 4) launch(k_vmm_mac<4, 1, 6>, 4, 4, 6);
    else if (r_o <= 8) launch(k_vmm_mac<4, 2, 3>, 4, 8, 3);
    else launch(k_vmm_mac<8, 2, 3>, 8, 16, 3);
}
// ---- masks before the shared rotations of query-times-K --------------------------------------------------
// A[k] = sum_{c < nk} T[c] * M[(c + k) mod E] for k < shared: T the nk key-ciphertext sums [2][limbs][n] (stacked),
// M the E slot rotations of the copy mask [E][limbs][n] (multiplier form), A stacked like T.  For one coefficient
// this is a correlation of the vector over c with the vector over the copies, so a lane that owns KO consecutive
// outputs k needs ONE new mask word per c: rows (c + k0) .. (c + k0 + KO - 1) slide by one.  A workgroup owns 64
// coefficients of one limb and stages CIRC_CC ciphertexts at a time in LDS (32 KiB); its four waves take KO outputs
// each.  Limbs below 2^50 multiply in FP64 (MacFp), the others in 128-bit integer sums reduced every 8 terms.
#define CIRC_CC 32
template <int KO>
__global__ __launch_bounds__(TPB) void k_mask_circulant(u64 *__restrict__ A, const u64 *__restrict__ T, const u64 *__restrict__ M,
                                                        const ModC *__restrict__ modc, const FpQ *__restrict__ fpq, int nk, int E,
                                                        int shared, int limbs, int n) {
    __shared__ u64 sb[CIRC_CC * 2 * MAC_CO];
    const int l = blockIdx.y, i0 = blockIdx.x * MAC_CO;
    const int co = threadIdx.x & (MAC_CO - 1), w = threadIdx.x >> 6;
    const int kb = (blockIdx.z * 4 + w) * KO;
    const bool active = kb < shared;
    const ModC m = modc[l];
    const FpQ fq = fpq[l];
    const bool fp = fq.q != 0.0;
    const MacFp F{fq.q, fq.qinv};
    const size_t cs = (size_t)limbs * n, ctw = 2 * cs, o = (size_t)l * n + i0;
    double s[KO][2];
    u64 v[KO][2];
#pragma unroll
    for (int t = 0; t < KO; t++) s[t][0] = s[t][1] = 0.0, v[t][0] = v[t][1] = 0;
    for (int c0 = 0; c0 < nk; c0 += CIRC_CC) {
        const int cn = nk - c0 < CIRC_CC ? nk - c0 : CIRC_CC;
        __syncthreads();
        {
            constexpr int ROWS = CIRC_CC * 2 * MAC_CO / TPB;      // all loads of a lane in flight before the first is used
            u64 x[ROWS];
#pragma unroll
            for (int it = 0; it < ROWS; it++) {
                const int jc = w + 4 * it;
                x[it] = jc < 2 * cn ? T[(size_t)(c0 + (jc >> 1)) * ctw + (jc & 1) * cs + o + co] : 0;
            }
#pragma unroll
            for (int it = 0; it < ROWS; it++) {
                const int jc = w + 4 * it;
                if (jc < 2 * cn) sb[jc * MAC_CO + co] = fp ? (u64)__double_as_longlong(MacFp::from_u64(x[it])) : x[it];
            }
        }
        __syncthreads();
        if (!active) continue;
        for (int c8 = 0; c8 < cn; c8 += 8) {
            u64 wv[KO + 7];
#pragma unroll
            for (int x = 0; x < KO + 7; x++)
                wv[x] = M[((size_t)((c0 + c8 + kb + x) & (E - 1)) * limbs + l) * n + i0 + co];     // E is a power of two
            if (fp) {
                double wa[KO + 7], waq[KO + 7];
#pragma unroll
                for (int x = 0; x < KO + 7; x++) wa[x] = MacFp::from_u64(wv[x]), waq[x] = wa[x] * F.qinv;
#pragma unroll
                for (int cc = 0; cc < 8; cc++) {
                    if (c8 + cc < cn) {
                        const double y0 = __longlong_as_double((long long)sb[((c8 + cc) * 2 + 0) * MAC_CO + co]);
                        const double y1 = __longlong_as_double((long long)sb[((c8 + cc) * 2 + 1) * MAC_CO + co]);
#pragma unroll
                        for (int t = 0; t < KO; t++) {
                            s[t][0] += F.mulmod(y0, wa[cc + t], waq[cc + t]);
                            s[t][1] += F.mulmod(y1, wa[cc + t], waq[cc + t]);
                        }
                    }
                    if ((cc & 3) == 3) {
#pragma unroll
                        for (int t = 0; t < KO; t++) s[t][0] = F.norm(s[t][0]), s[t][1] = F.norm(s[t][1]);
                    }
                }
            } else {
                u128 a[KO][2];
#pragma unroll
                for (int t = 0; t < KO; t++) a[t][0] = a[t][1] = 0;
#pragma unroll
                for (int cc = 0; cc < 8; cc++) {
                    if (c8 + cc < cn) {
                        const u64 y0 = sb[((c8 + cc) * 2 + 0) * MAC_CO + co], y1 = sb[((c8 + cc) * 2 + 1) * MAC_CO + co];
#pragma unroll
                        for (int t = 0; t < KO; t++) a[t][0] += (u128)y0 * wv[cc + t], a[t][1] += (u128)y1 * wv[cc + t];
                    }
                }
#pragma unroll
                for (int t = 0; t < KO; t++) {
                    v[t][0] = addmod(v[t][0], redc(a[t][0], m.q, m.qinv), m.q);
                    v[t][1] = addmod(v[t][1], redc(a[t][1], m.q, m.qinv), m.q);
                }
            }
        }
    }
    if (!active) return;
#pragma unroll
    for (int t = 0; t < KO; t++) {
        if (kb + t < shared) {
            u64 *dst = A + (size_t)(kb + t) * ctw + o + co;
            dst[0] = fp ? F.canon(F.mulmod(s[t][0], fq.rinv, fq.rinvq)) : v[t][0];
            dst[cs] = fp ? F.canon(F.mulmod(s[t][1], fq.rinv, fq.rinvq)) : v[t][1];
        }
    }
}
void launch_mask_circulant(cm_ctx *ctx, u64 *A, const u64 *T, const u64 *M, int nk, int E, int shared, int limbs, hipStream_t st) {
    Prof prof_(ctx, CM_K_ELEMENTWISE, (double)nk * shared * 2 * limbs, st);
    const int ko = shared >= 8 ? 8 : shared >= 4 ? 4 : 2;
    const dim3 grid(ctx->n / MAC_CO, limbs, (shared + 4 * ko - 1) / (4 * ko)), block(TPB);
    if (ko == 8)
        hipLaunchKernelGGL(k_mask_circulant<8>, grid, block, 0, st, A, T, M, ctx->d_modc, ctx->d_fpq, nk, E, shared, limbs, ctx->n);
    else if (ko == 4)
        hipLaunchKernelGGL(k_mask_circulant<4>, grid, block, 0, st, A, T, M, ctx->d_modc, ctx->d_fpq, nk, E, shared, limbs, ctx->n);
    else
        hipLaunchKernelGGL(k_mask_circulant<2>, grid, block, 0, st, A, T, M, ctx->d_modc, ctx->d_fpq, nk, E, shared, limbs, ctx->n);
}
// The same sums through a length-E transform along the copy index: for one coefficient A[k] = sum_c t[c] m[(c + k) mod E]
// is a cyclic correlation, so with t'[c] = t[(-c) mod E] and F the length-E number-theoretic transform (E divides
// q - 1), A = F^-1( F(m) . F(t') ): E (log2 E + 1) products per coefficient instead of nk * shared, exact like the direct sum.
// MODE 0 (set-up): rows M[E][limbs][n] -> Mhat = F(m) / E, kept in the order the forward pass leaves (bit-reversed), in
// multiplier form (nk != 0) or as plain residues (nk = 0);
// MODE 1: T[nk] stacked ciphertexts -> A[shared].  A workgroup owns CO coefficients of one limb and one component and
// keeps the E x CO words in LDS; the forward pass is decimation in frequency, the inverse one decimation in time, so
// no reordering is needed.  tw[limbs][2][E/2][2]: omega^e and omega^-e with their companions; einv[limbs]: E^-1 in
// multiplier form.
template <int MODE>
__global__ __launch_bounds__(TPB) void k_mask_ntt(u64 *__restrict__ out, const u64 *__restrict__ in, const u64 *__restrict__ Mhat,
                                                  const u64 *__restrict__ tw, const u64 *__restrict__ einv,
                                                  const ModC *__restrict__ modc, int nk, int E, int logE, int shared, int limbs,
                                                  int n, int logCO) {
    extern __shared__ u64 X[];
    const int CO = 1 << logCO, l = blockIdx.y, comp = blockIdx.z, i0 = blockIdx.x * CO;
    const ModC m = modc[l];
    const u64 q = m.q;
    const size_t cs = (size_t)limbs * n, ctw = 2 * cs, o = (size_t)l * n + i0;
    for (int e = threadIdx.x; e < E * CO; e += TPB) {
        const int c = e >> logCO, co = e & (CO - 1);
        if (MODE == 1) X[(((E - c) & (E - 1)) << logCO) + co] = c < nk ? in[(size_t)c * ctw + comp * cs + o + co] : 0;
        else X[e] = in[(size_t)c * cs + o + co];
    }
    __syncthreads();
    const u64 *twf = tw + (size_t)l * 2 * E, *twi = twf + E;
    for (int lg = logE - 1; lg >= 0; lg--) {                       // half-length 2^lg, twiddle step 2^(logE - 1 - lg)
        const int len = 1 << lg, sh = logE - 1 - lg;
        for (int id = threadIdx.x; id < (E / 2) * CO; id += TPB) {
            const int bf = id >> logCO, co = id & (CO - 1), j = bf & (len - 1);
            const int a = ((((bf >> lg) << (lg + 1)) + j) << logCO) + co, b = a + (len << logCO);
            const u64 u = X[a], v = X[b];
            X[a] = addmod(u, v, q);
            const int e = j << sh;
            X[b] = mul_shoup(submod(u, v, q), twf[2 * e], twf[2 * e + 1], q);
        }
        __syncthreads();
    }
    if (MODE == 0) {
        const u64 s = einv[l];
        for (int e = threadIdx.x; e < E * CO; e += TPB) {
            const u64 x = redc((u128)X[e] * s, q, m.qinv);
            out[(size_t)(e >> logCO) * cs + o + (e & (CO - 1))] = nk ? x : redc((u128)x, q, m.qinv);
        }
        return;
    }
    for (int e = threadIdx.x; e < E * CO; e += TPB)
        X[e] = redc((u128)X[e] * Mhat[(size_t)(e >> logCO) * cs + o + (e & (CO - 1))], q, m.qinv);
    __syncthreads();
    for (int lg = 0; lg < logE; lg++) {
        const int len = 1 << lg, sh = logE - 1 - lg;
        for (int id = threadIdx.x; id < (E / 2) * CO; id += TPB) {
            const int bf = id >> logCO, co = id & (CO - 1), j = bf & (len - 1);
            const int a = ((((bf >> lg) << (lg + 1)) + j) << logCO) + co, b = a + (len << logCO);
            const int e = j << sh;
            const u64 u = X[a], v = mul_shoup(X[b], twi[2 * e], twi[2 * e + 1], q);
            X[a] = addmod(u, v, q);
            X[b] = submod(u, v, q);
        }
        __syncthreads();
    }
    for (int e = threadIdx.x; e < shared * CO; e += TPB)
        out[(size_t)(e >> logCO) * ctw + comp * cs + o + (e & (CO - 1))] = X[e];
}
// The same sums on limbs below 2^50 in FP64 and registers, for E = 2^(L1 + L2) = 16 .. 256: a lane holds 2^L1 rows of one
// coefficient, the forward pass is L1 stages, an exchange through LDS and L2 stages; the product with Mhat and the first L2
// inverse stages happen on the same registers, one more exchange, L1 stages.  The workgroups of the two components are
// neighbours, so that Mhat comes from HBM about once.
// Bound by memory (T and A once, Mhat once): the integer form above walks through LDS and a barrier at every one of its
// 2 log2 E stages.  Measured, 126 ciphertexts of 12 limbs, E = 128: 3.69 -> 1.11 ms (4 GB; with
// both components in one workgroup and its Mhat words kept over them 1.52 ms, two waves a SIMD).
// Bounds in units of q (products: 1/2 + 3/8 B): forward sums are renormalised, differences stay below 4, products below 2;
// from the product with Mhat (1.25, renormalised where L2 = 4) three inverse stages reach 5.4, are renormalised, and four
// or fewer more reach 5.2.
template <int L1, int L2>
__global__ __launch_bounds__(TPB) void k_mask_ntt_fp(u64 *__restrict__ out, const u64 *__restrict__ in, const u64 *__restrict__ Mhat,
                                                     const u64 *__restrict__ tw, const FpQ *__restrict__ fpq, int nk, int shared,
                                                     int limbs, int n) {
    constexpr int E = 1 << (L1 + L2), NV = 1 << L1, NB = 1 << (L1 - L2), BL = 1 << L2, CO = TPB >> L2;
    __shared__ double X[E * CO];
    __shared__ double wt[2][E / 2];
    const int l = blockIdx.y, comp = blockIdx.x & 1, i0 = (blockIdx.x >> 1) * CO, co = threadIdx.x & (CO - 1), s = threadIdx.x / CO;
    const FpQ fq = fpq[l];
    const MacFp F{fq.q, fq.qinv};
    const size_t cs = (size_t)limbs * n, ctw = 2 * cs, o = (size_t)l * n + i0 + co;
    for (int e = threadIdx.x; e < E; e += TPB) wt[e / (E / 2)][e % (E / 2)] = MacFp::from_u64(tw[(size_t)l * 2 * E + 2 * e]);
    double v[NV];
    {
        u64 raw[NV];
#pragma unroll
        for (int k = 0; k < NV; k++) {
            const int c = (E - (k * BL + s)) & (E - 1);
            raw[k] = c < nk ? __builtin_nontemporal_load(in + (size_t)c * ctw + comp * cs + o) : 0;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NV; k++) v[k] = MacFp::from_u64(raw[k]);
    }
    // forward, decimation in frequency: rows k BL + s
#pragma unroll
    for (int a = 0; a < L1; a++) {
        const int half = NV >> (a + 1);
#pragma unroll
        for (int j = 0; j < half; j++) {
            const double w = wt[0][(j * BL + s) << a], wq = w * F.qinv;
#pragma unroll
            for (int g = 0; g < (1 << a); g++) {
                const int k = g * 2 * half + j;
                const double u = v[k], y = v[k + half];
                v[k] = F.norm(u + y), v[k + half] = F.mulmod(u - y, w, wq);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < NV; k++) X[(k * BL + s) * CO + co] = v[k];
    u64 mh[NV];                               // in flight across the exchange
#pragma unroll
    for (int x = 0; x < NV; x++) mh[x] = Mhat[(size_t)((s * NB + x / BL) * BL + x % BL) * cs + o];
    __syncthreads();
    // rows (s NB + b) BL + k
#pragma unroll
    for (int x = 0; x < NV; x++) v[x] = X[((s * NB + x / BL) * BL + x % BL) * CO + co];
#pragma unroll
    for (int a = 0; a < L2; a++) {
        const int half = BL >> (a + 1);
#pragma unroll
        for (int j = 0; j < half; j++) {
            const double w = wt[0][j << (L1 + a)], wq = w * F.qinv;
#pragma unroll
            for (int g = 0; g < (NB << a); g++) {
                const int k = g * 2 * half + j;
                const double u = v[k], y = v[k + half];
                v[k] = F.norm(u + y), v[k + half] = F.mulmod(u - y, w, wq);
            }
        }
    }
#pragma unroll
    for (int x = 0; x < NV; x++) {
        const double m = MacFp::from_u64(mh[x]);
        v[x] = F.mulmod(v[x], m, m * F.qinv);
        if (L2 > 3) v[x] = F.norm(v[x]);
    }
    // inverse, decimation in time
#pragma unroll
    for (int a = L2 - 1; a >= 0; a--) {
        const int half = BL >> (a + 1);
#pragma unroll
        for (int j = 0; j < half; j++) {
            const double w = wt[1][j << (L1 + a)], wq = w * F.qinv;
#pragma unroll
            for (int g = 0; g < (NB << a); g++) {
                const int k = g * 2 * half + j;
                const double u = v[k], y = F.mulmod(v[k + half], w, wq);
                v[k] = u + y, v[k + half] = u - y;
            }
        }
    }
#pragma unroll
    for (int x = 0; x < NV; x++) X[((s * NB + x / BL) * BL + x % BL) * CO + co] = F.norm(v[x]);       // the words it read
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; k++) v[k] = X[(k * BL + s) * CO + co];
#pragma unroll
    for (int a = L1 - 1; a >= 0; a--) {
        const int half = NV >> (a + 1);
#pragma unroll
        for (int j = 0; j < half; j++) {
            const double w = wt[1][(j * BL + s) << a], wq = w * F.qinv;
#pragma unroll
            for (int g = 0; g < (1 << a); g++) {
                const int k = g * 2 * half + j;
                const double u = v[k], y = F.mulmod(v[k + half], w, wq);
                v[k] = u + y, v[k + half] = u - y;
            }
        }
    }
#pragma unroll
    for (int k = 0; k < NV; k++) {
        const int c = k * BL + s;
        if (c < shared) __builtin_nontemporal_store(F.canon(v[k]), out + (size_t)c * ctw + comp * cs + o);
    }
}
// where the FP64 form runs (its Mhat is kept as plain residues, the integer form's in multiplier form)
static bool mask_ntt_fp(const cm_ctx *ctx, int E, int limbs) {
    bool fp = E >= 16 && E <= 256;
    for (int l = 0; l < limbs; l++) fp = fp && ctx->mod[l] < (1ULL << 50);
    return fp;
}
// CO = min(64, 4096 / E) coefficients per workgroup (32 KiB of LDS at most); 8 <= E <= 512
static int mask_ntt_log_co(int E) {
    int lg = 6;
    while ((E << lg) > 4096) lg--;
    return lg;
}
bool mask_ntt_supported(int E) { return E >= 8 && E <= 512 && (E & (E - 1)) == 0; }
void launch_mask_ntt_setup(cm_ctx *ctx, u64 *Mhat, const u64 *M, const u64 *tw, const u64 *einv, int E, int limbs, hipStream_t st) {
    int logE = 0;
    while ((1 << logE) < E) logE++;
    const int lg = mask_ntt_log_co(E);
    hipLaunchKernelGGL(k_mask_ntt<0>, dim3(ctx->n >> lg, limbs, 1), dim3(TPB), ((size_t)E << lg) * 8, st, Mhat, M, nullptr, tw, einv,
                       ctx->d_modc, mask_ntt_fp(ctx, E, limbs) ? 0 : E, E, logE, E, limbs, ctx->n, lg);
}
void launch_mask_ntt(cm_ctx *ctx, u64 *A, const u64 *T, const u64 *Mhat, const u64 *tw, const u64 *einv, int nk, int E, int shared,
                     int limbs, hipStream_t st) {
    Prof prof_(ctx, CM_K_ELEMENTWISE, (double)E * 2 * limbs, st);
    int logE = 0;
    while ((1 << logE) < E) logE++;
    if (mask_ntt_fp(ctx, E, limbs)) {
#define MASK_FP(L1_, L2_)                                                                                                        \
    hipLaunchKernelGGL((k_mask_ntt_fp<L1_, L2_>), dim3(2 * ctx->n / (TPB >> L2_), limbs), dim3(TPB), 0, st, A, T, Mhat, tw, ctx->d_fpq, nk, \
                       shared, limbs, ctx->n)
        if (logE == 4) MASK_FP(2, 2);
        else if (logE == 5) MASK_FP(3, 2);
        else if (logE == 6) MASK_FP(3, 3);
        else if (logE == 7) MASK_FP(4, 3);
        else MASK_FP(4, 4);
#undef MASK_FP
        return;
    }
    const int lg = mask_ntt_log_co(E);
    hipLaunchKernelGGL(k_mask_ntt<1>, dim3(ctx->n >> lg, limbs, 2), dim3(TPB), ((size_t)E << lg) * 8, st, A, T, Mhat, tw, einv,
                       ctx->d_modc, nk, E, logE, shared, limbs, ctx->n, lg);
}
// plaintext (j,k) between its plain form src[limbs][n] and its place in the blocked array.  The words of a packed group share
// some bits' places: a launch writes one plaintext, so a lane reads and writes the places of its coefficient alone.
__global__ void k_pt_block(u64 *blocked, u64 *plain, MacLayout lay, int n, int j, int k, int to_blocked) {
    const int i = blockIdx.x * TPB + threadIdx.x, l = blockIdx.y, co = i % MAC_CO;
    u64 *grp = blocked + lay.group(l, i / MAC_CO, j / lay.per_group(), k);
    const int jj = j % lay.per_group();
    const size_t p = (size_t)l * n + i;
    unsigned *dw = (unsigned *)grp;
    if (lay.is50(l)) {
        unsigned *lo = dw + (jj / 4) * 256 + co * 4 + (jj & 3);
        unsigned short *mid = (unsigned short *)(dw + 512) + co * 8 + jj, *top = (unsigned short *)(dw + 768) + co;
        if (to_blocked) {
            const u64 v = plain[p];
            *lo = (unsigned)v, *mid = (unsigned short)(v >> 32);
            *top = (unsigned short)((*top & ~(3u << (2 * jj))) | ((unsigned)(v >> 48) << (2 * jj)));
        } else {
            plain[p] = (u64)*lo | ((u64)*mid << 32) | ((u64)((*top >> (2 * jj)) & 3u) << 48);
        }
    } else if (lay.is60(l)) {
        auto d = [&](int i) -> unsigned & { return i < 12 ? dw[(i / 4) * 256 + co * 4 + i % 4] : dw[768 + co * 3 + i % 4]; };
        auto put = [&](int h, unsigned v) {
            if (h < 15) d(h) = (d(h) & ~LOW30) | v;
            else for (int i = 0; i < 15; i++) d(i) = (d(i) & LOW30) | (((v >> (28 - 2 * i)) & 3u) << 30);
        };
        auto get = [&](int h) {
            unsigned v = 0;
            if (h < 15) v = d(h) & LOW30;
            else for (int i = 0; i < 15; i++) v = (v << 2) | (d(i) >> 30);
            return v;
        };
        if (to_blocked) put(2 * jj, (unsigned)plain[p] & LOW30), put(2 * jj + 1, (unsigned)(plain[p] >> 30));
        else plain[p] = (u64)get(2 * jj) | ((u64)get(2 * jj + 1) << 30);
    } else {
        const int b = lay.word(jj, co);
        if (to_blocked) grp[b] = plain[p];
        else plain[p] = grp[b];
    }
}
void launch_pt_block(cm_ctx *ctx, u64 *blocked, u64 *plain, int limbs, int level, int r_i, int r_o, int j, int k, bool to_blocked,
                     hipStream_t st) {
    hipLaunchKernelGGL(k_pt_block, dim3(ctx->n / TPB, limbs), dim3(TPB), 0, st, blocked, plain, mac_layout(ctx, r_i, r_o, limbs, level),
                       ctx->n, j, k, to_blocked ? 1 : 0);
}
