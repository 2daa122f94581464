// Rotary position embedding with the ciphertext extraction fused into it (Sec. 4.2, App. D).
//
// A projection leaves partial sums in every slot that is not an output slot; the element-wise
// layer that follows multiplies by plaintexts that are zero there, so the clean-up costs no level
// of its own.  For q and k that layer is the rotary embedding: with the head-interleaved layout
// slot (e, h, tau) = (e*H + h)*t + tau of Sec. 5.3, the dims 2m and 2m+1 of a head sit H*t slots
// apart, and for token n
//     p0 = cos(theta) on the valid slots,  p1 = sin(theta) on those of even dims,
//     p2 = -sin(theta) on those of odd dims,            theta = n * base^(-2m/E),
//     y  = x p0 + Rot(x p2, +H t) + Rot(x p1, -H t)      (three products, two rotations, one level).
// The appendix prints the single-head case ("rotate by 1" = one block); the signs are read so that
// they fit the left-rotation convention of Sec. 2.1.  The plaintexts are encoded at the scale of
// the prime that the rescale removes, so the ciphertext keeps its scale.
#include <math.h>

#include "kernels.h"

struct cm_rope {
    cm_ctx *ctx = nullptr;
    int S, H, E, t, level, token, tau;
    int step_up, step_dn;      // y = x p0 + Rot(x p2, step_up) + Rot(x p1, step_dn)
    double base;
    u64 *d_pts = nullptr;      // [3][level+1][n], multiplier form
    u64 *d_work = nullptr;     // three ciphertexts
    KsManyTables tabs;         // raise of the two rotated second components at once
};

static bool pow2(int x) { return x > 0 && (x & (x - 1)) == 0; }

// out_k = a * pt_k for k = 0, 1, 2: the ciphertext is read once
__global__ void k_mul_pt3(u64 *out0, u64 *out1, u64 *out2, const u64 *__restrict__ a, const u64 *__restrict__ pts,
                          const ModC *__restrict__ modc, int limbs, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x, r = blockIdx.y, l = r % limbs;
    const ModC m = modc[l];
    const size_t o = (size_t)r * n + i, po = (size_t)l * n + i, ps = (size_t)limbs * n;
    const u64 v = a[o];
    out0[o] = redc((u128)v * pts[po], m.q, m.qinv);
    out1[o] = redc((u128)v * pts[ps + po], m.q, m.qinv);
    out2[o] = redc((u128)v * pts[2 * ps + po], m.q, m.qinv);
}

// The same products, the second and third already rotated (read through their Galois maps) and, of the first components,
// summed: sum[2][limbs][n] = (a0 p0 + sigma_u(a0 p2) + sigma_d(a0 p1), a1 p0), rot[2][limbs][n] = sigma_u(a1 p2), sigma_d(a1 p1)
__global__ void k_mul_pt3_rot(u64 *__restrict__ sum, u64 *__restrict__ rot, const u64 *__restrict__ a, const u64 *__restrict__ pts,
                              const ModC *__restrict__ modc, int limbs, int n, int logn, unsigned gu, unsigned gd) {
    const unsigned i = blockIdx.x * 256 + threadIdx.x, iu = perm_src(i, gu, logn), id = perm_src(i, gd, logn);
    const int r = blockIdx.y, l = r % limbs;
    const ModC m = modc[l];
    const size_t row = (size_t)r * n, po = (size_t)l * n, ps = (size_t)limbs * n;
    const u64 v = redc((u128)a[row + i] * pts[po + i], m.q, m.qinv);
    const u64 u = redc((u128)a[row + iu] * pts[2 * ps + po + iu], m.q, m.qinv);
    const u64 d = redc((u128)a[row + id] * pts[ps + po + id], m.q, m.qinv);
    if (r < limbs) {
        sum[row + i] = addmod(addmod(v, u, m.q), d, m.q);
    } else {
        sum[row + i] = v;
        rot[po + i] = u;
        rot[ps + po + i] = d;
    }
}

extern "C" cm_status cm_rope_create(cm_ctx *ctx, int32_t heads, int32_t dim, int32_t level, int32_t token, int32_t tau,
                                    double base, const int64_t *coeffs, cm_rope **out) {
    if (!ctx || !out || heads < 1 || dim < 2 || token < 0 || !(base > 1.0)) return CM_E_INVAL;
    if (level < 1 || level > ctx->L) return CM_E_LEVEL;
    const int S = ctx->n / 2;
    while (!pow2(heads)) heads++;          // a head count that is not a power of two is padded to the next one
    if (!pow2(dim) || heads * dim > S) return CM_E_LAYOUT;
    const int t = S / (heads * dim);
    if (tau < -1 || tau >= t) return CM_E_LAYOUT;
    cm_rope *r = new (std::nothrow) cm_rope();
    if (!r) return CM_E_NOMEM;
    try {
    r->ctx = ctx, r->S = S, r->H = heads, r->E = dim, r->t = t, r->level = level, r->token = token, r->tau = tau, r->base = base;
    r->step_up = heads * t, r->step_dn = -(heads * t);
    const size_t n = ctx->n, ln = (size_t)(level + 1) * n;
    if (hipMalloc((void **)&r->d_pts, 3 * ln * 8) != hipSuccess || hipMalloc((void **)&r->d_work, 6 * ln * 8) != hipSuccess) {
        cm_rope_destroy(r);
        return CM_E_NOMEM;
    }
    if (ks_many_tables_create(ctx, level, 2, &r->tabs, 1, 0) != CM_OK) {
        cm_rope_destroy(r);
        return CM_E_NOMEM;
    }
    const double scale = (double)ctx->mod[level];
    cm_status s = CM_OK;
    std::vector<double> p[3];
    for (auto &v : p) v.assign(S, 0.0);
    // tau = -1: a group of t tokens, token + r at residue r
    for (int r0 = (tau < 0 ? 0 : tau); r0 < (tau < 0 ? t : tau + 1) && !coeffs; r0++)
        for (int e = 0; e < dim; e++) {
            const double th = (double)(token + (tau < 0 ? r0 : 0)) * pow(base, -2.0 * (double)(e / 2) / (double)dim);
            for (int h = 0; h < heads; h++) {
                const size_t i = ((size_t)e * heads + h) * t + r0;
                p[0][i] = cos(th);
                if (e % 2 == 0) p[1][i] = sin(th);
                else p[2][i] = -sin(th);
            }
        }
    for (int k = 0; k < 3 && s == CM_OK; k++) {
        cm_pt pt;
        pt.dev = r->d_pts + k * ln, pt.mont = 1;
        s = coeffs ? cm_pt_from_coeffs(ctx, coeffs + (size_t)k * n, level, scale, &pt)
                   : cm_encode(ctx, p[k].data(), nullptr, p[k].size(), level, scale, &pt);
    }
    if (s != CM_OK) { cm_rope_destroy(r); return s; }
    *out = r;
    return CM_OK;
    } catch (...) {
        cm_rope_destroy(r);
        return CM_E_NOMEM;
    }
}
// Inner rotation (Sec. 5.4): residue tau of every block of t slots moves to residue (tau + delta) mod t.  The same
// shape as the embedding: p0 = 0, p2 = the residues below t - delta (rotated by -delta), p1 = the others (rotated by
// t - delta); masks encoded at the scale of the prime the rescale removes.
extern "C" cm_status cm_inner_rot_create(cm_ctx *ctx, int32_t t, int32_t delta, int32_t level, const int64_t *coeffs,
                                         cm_rope **out) {
    if (!ctx || !out) return CM_E_INVAL;
    if (level < 1 || level > ctx->L) return CM_E_LEVEL;
    const int S = ctx->n / 2;
    if (!pow2(t) || t < 2 || t > S || delta < 1 || delta >= t) return CM_E_LAYOUT;
    cm_rope *r = new (std::nothrow) cm_rope();
    if (!r) return CM_E_NOMEM;
    try {
    r->ctx = ctx, r->S = S, r->H = 1, r->E = S / t, r->t = t, r->level = level, r->token = 0, r->tau = 0, r->base = 0;
    r->step_up = -delta, r->step_dn = t - delta;
    const size_t n = ctx->n, ln = (size_t)(level + 1) * n;
    if (hipMalloc((void **)&r->d_pts, 3 * ln * 8) != hipSuccess || hipMalloc((void **)&r->d_work, 6 * ln * 8) != hipSuccess) {
        cm_rope_destroy(r);
        return CM_E_NOMEM;
    }
    if (ks_many_tables_create(ctx, level, 2, &r->tabs, 1, 0) != CM_OK) {
        cm_rope_destroy(r);
        return CM_E_NOMEM;
    }
    const double scale = (double)ctx->mod[level];
    std::vector<double> p[3];
    for (auto &v : p) v.assign(S, 0.0);
    for (int i = 0; i < S && !coeffs; i++) p[(i % t) < t - delta ? 2 : 1][i] = 1.0;
    cm_status s = CM_OK;
    for (int k = 0; k < 3 && s == CM_OK; k++) {
        cm_pt pt;
        pt.dev = r->d_pts + k * ln, pt.mont = 1;
        s = coeffs ? cm_pt_from_coeffs(ctx, coeffs + (size_t)k * n, level, scale, &pt)
                   : cm_encode(ctx, p[k].data(), nullptr, p[k].size(), level, scale, &pt);
    }
    if (s != CM_OK) { cm_rope_destroy(r); return s; }
    *out = r;
    return CM_OK;
    } catch (...) {
        cm_rope_destroy(r);
        return CM_E_NOMEM;
    }
}
extern "C" void cm_rope_destroy(cm_rope *r) {
    if (!r) return;
    ks_many_tables_destroy(&r->tabs);
    hipFree(r->d_pts);
    hipFree(r->d_work);
    delete r;
}
extern "C" int32_t cm_rope_steps(const cm_rope *r, int32_t *steps, int32_t cap) {
    if (!r) return 0;
    const int s[2] = {r->step_up, r->step_dn};
    for (int i = 0; i < 2 && i < cap && steps; i++) steps[i] = s[i];
    return 2;
}
extern "C" cm_status cm_rope_apply(cm_ctx *ctx, const cm_evk *evk, const cm_rope *r, const cm_ct *x, cm_ct *y, void *stream) {
    (void)hipGetLastError();          // stale errors of earlier calls are not this call's
    if (!ctx || !evk || !r || r->ctx != ctx || !x || !x->dev || x->ncomp != 2 || !y || !y->dev || y->dev == x->dev ||
        !evk_fits(ctx, evk))
        return CM_E_INVAL;
    if (x->level != r->level) return CM_E_LEVEL;
    CM_TRY
    hipStream_t st = (hipStream_t)stream;
    const int level = r->level, limbs = level + 1;
    const u64 g_up = galois_of_step(ctx, r->step_up), g_dn = galois_of_step(ctx, r->step_dn);
    const u64 *k_up = find_key(evk, g_up), *k_dn = find_key(evk, g_dn);
    if (!k_up || !k_dn) return CM_E_NOKEY;
    const size_t n = ctx->n, ctw = 2 * (size_t)limbs * n;
    u64 *a = r->d_work, *b = a + ctw, *c = b + ctw;
    const KsLevel &kl = ks_level(ctx, level);
    const size_t dblk = (size_t)kl.beta * kl.ext * n;
    if (ks_drop_fits(ctx, level, 2, 1) && 2 * dblk <= arena_digits_words(ctx)) {
        // Both rotations and the rescale in one go, ten launches instead of twenty-three (each takes its 4 to 8 us at the low
        // levels): products rotated as they are formed, one raise and one inner product for both, and since the two ModDowns
        // and the rescale are sums of conversions, one forward transform for all of them (ks_drop with two sets).
        u64 *digits = arena_digits(ctx);
        hipLaunchKernelGGL(k_mul_pt3_rot, dim3(n / 256, 2 * limbs), dim3(256), 0, st, a, b, x->dev, r->d_pts, ctx->d_modc, limbs, (int)n,
                           ctx->logn, (unsigned)g_up, (unsigned)g_dn);
        const bool half = rows_ip_fits(ctx, kl.beta, level, 1, 2);
        CMCHK(ks_raise_many(ctx, r->tabs, b, c, digits, st, -1, 0, half));
        IpBatch ip;
        ip.nz = 1, ip.nsum = 2, ip.apart = true;
        ip.it[0].dig = digits, ip.it[0].key = k_up, ip.it[1].dig = digits + dblk, ip.it[1].key = k_dn;
        ip.out[0] = arena_batch_sums(ctx);
        ip.it[0].own = b, ip.it[1].own = b + (size_t)limbs * n;
        if (half) launch_rows_ip(ctx, ip, kl.beta, level, st, level, ks_drop_fold(ctx, level, 2, nullptr, 0, 0, 0, a, 0));
        else launch_inner_product_batch(ctx, ip, kl.beta, level, st);
        CMCHK(ks_drop(ctx, ip.out[0], level, 2, 1, nullptr, 0, 0, 0, a, 0, y->dev, st, half));
        y->level = level - 1, y->ncomp = 2;
        y->scale = x->scale;                                      // plaintext scale = the prime just removed
        RETURN_LAUNCH_STATUS();
    }
    hipLaunchKernelGGL(k_mul_pt3, dim3(ctx->n / 256, 2 * limbs), dim3(256), 0, st, a, c, b, x->dev, r->d_pts, ctx->d_modc, limbs,
                       ctx->n);                                   // a = x p0, c = x p1, b = x p2
    CMCHK(rotate_into(ctx, k_up, b, level, g_up, a, st, a));      // a += Rot(x p2, step_up)
    CMCHK(rotate_into(ctx, k_dn, c, level, g_dn, a, st, a));      // a += Rot(x p1, step_dn)
    CMCHK(rescale_into(ctx, a, 2, level, y->dev, st));
    y->level = level - 1, y->ncomp = 2;
    y->scale = x->scale;                                          // plaintext scale = the prime just removed
    RETURN_LAUNCH_STATUS();
    CM_CATCH
}
