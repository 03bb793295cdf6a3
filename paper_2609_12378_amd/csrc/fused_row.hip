// Steps that end in a forward transform, for N >= 2^12 (rows of 256 points) in either arithmetic: the element-wise
// work that follows the transform runs in its row pass, and the element-wise work before it in the column pass, so
// the transformed rows never go to HBM on their own.  A rescale is four launches (it was eight), an encryption or a
// decryption two (five).
//
//   rescale     out_i = (c_i - NTT(top mod q_i)) q_l^-1, top the centred coefficients of the top limb
//   ModDown     out_i = (u_i - NTT(conv)) P^-1 + addend            (integer arithmetic; fp64 has k_ks_finish8)
//   decryption  pt = c0 + c1 NTT(s)
//   encryption  (c0, c1) = (NTT(e) + m - a NTT(s), a)
#include <algorithm>

#include "ckks_internal.h"
#include "ks_args.h"
#include "ops.h"

namespace {

using nttc::Ar;
using nttc::kE;

template <bool F>
using E = typename Ar<F>::E;
template <bool F>
using W = typename Ar<F>::W;

template <bool F>
__device__ __forceinline__ const W<F> *table(const void *t, uint32_t prime, uint32_t log_n)
{
    return (const W<F> *)t + ((size_t)prime << log_n);
}

// forward row masks: fp64 column passes leave rows below 4.3 q; stages 0, 2, 4, 6 reducing keep every value below 7 q
// and the output below 4 q
constexpr unsigned kRowMask = 0x55;

// forward row pass of row h, in registers: x[k] is point t + 16 k in and out (lds: this row's 273 words)
template <bool F>
__device__ __forceinline__ void row_forward(E<F> (&x)[kE], E<F> *lds, const W<F> *tw, uint32_t B, uint32_t sub,
                                            uint32_t t, const Ar<F> &ar)
{
    nttc::fwd_top<F, kRowMask>(x, tw, B, ar);
    nttc::transpose<8, true>(x, lds, sub, t);
    nttc::fwd_low<8, F, kRowMask>(x, tw, B, t, ar);
    nttc::transpose<8, false>(x, lds, sub, t);
}

// the transformed value and a canonical residue v combined: (v - x) w (w canonical, ws its Shoup companion) as a lazy
// value, then canonical sums
__device__ __forceinline__ uint64_t sub_mul(const Ar<true> &ar, uint64_t v, double x, ulonglong2 w, uint64_t add)
{
    return ar.to_canon(ar.mul(Ar<true>::from_u64(v) - x, (double)w.x) + Ar<true>::from_u64(add));
}
__device__ __forceinline__ uint64_t sub_mul(const Ar<false> &ar, uint64_t v, uint64_t x, ulonglong2 w, uint64_t add)
{
    return addmod(shoup(submod(v, ar.to_canon(x), ar.q), w.x, w.y, ar.q), add, ar.q);
}

enum { FIN_RESCALE = 0, FIN_MODDOWN = 1 };

struct FinArgs {
    const uint64_t *in;        // rows after the column pass [polys][limbs][N]
    const uint64_t *c;         // rescale: [polys][limbs + 1][N]; ModDown: u [polys][u_rows][N]
    uint64_t *out;             // rescale: [polys][limbs][N]; null: polynomial p to ra.out[p / 2], component p % 2
    uint32_t limbs, c_rows, polys, log_n;
    const ulonglong2 *w;       // [limbs]
};

// 8 rows of one limb per block of 128 threads: rows 8 blk .. of one polynomial, or (SHARE, polys a multiple of 8) the
// same row of 8 polynomials, which then read one row of twiddles (the integer arithmetic's pairs are 16 bytes a
// butterfly group)
template <bool F, int FIN, bool SHARE>
__global__ __launch_bounds__(128) void k_row_fin(FinArgs a, RotArgs ra, const ModQ *__restrict__ mods,
                                                 const void *__restrict__ tw_all)
{
    __shared__ E<F> lds[8 * 273];
    const uint32_t n1 = 1u << (a.log_n - 8), sub = threadIdx.x >> 4, t = threadIdx.x & 15u;
    uint32_t h, l, p;
    if (SHARE) {
        h = blockIdx.x % n1;
        const uint32_t rest = blockIdx.x / n1;
        l = rest % a.limbs;
        p = 8 * (rest / a.limbs) + sub;
    } else {
        const uint32_t per = n1 / 8, row = blockIdx.x / per;
        h = (blockIdx.x % per) * 8 + sub;
        l = row % a.limbs;
        p = row / a.limbs;
    }
    const Ar<F> ar(mods[l]);
    const size_t off = (size_t)h * 256;
    const uint64_t *in = a.in + (((size_t)p * a.limbs + l) << a.log_n) + off;
    const uint64_t *c = a.c + (((size_t)p * a.c_rows + l) << a.log_n) + off;
    E<F> x[kE];
    uint64_t cv[kE];
#pragma unroll
    for (int k = 0; k < kE; k++) x[k] = ar.from_raw(nttc::ld_stream(in + t + 16 * k));
#pragma unroll
    for (int k = 0; k < kE; k++) cv[k] = nttc::ld_stream(c + t + 16 * k);
    row_forward<F>(x, lds, table<F>(tw_all, l, a.log_n), n1 + h, sub, t, ar);
    const ulonglong2 w = a.w[l];
    if constexpr (FIN == FIN_RESCALE) {
        uint64_t *out = (a.out ? a.out + ((size_t)p * a.limbs << a.log_n)
                               : ra.out[p >> 1] + ((size_t)(p & 1) * a.limbs << a.log_n)) + ((size_t)l << a.log_n) + off;
#pragma unroll
        for (int k = 0; k < kE; k++) nttc::st_stream(out + t + 16 * k, sub_mul(ar, cv[k], x[k], w, 0));
    } else {
        // polynomial p is component p % 2 of rotation p / 2
        const uint32_t r = p >> 1, comp = p & 1;
        uint64_t *out = ra.out[r] + (((size_t)comp * a.limbs + l) << a.log_n) + off;
        const uint64_t *add = comp ? ra.add1[r] : ra.c0[r];
        const uint32_t g = comp ? 1u : ra.g[r];
#pragma unroll
        for (int k = 0; k < kE; k++) {
            const uint32_t pos = (uint32_t)off + t + 16 * k;
            const uint64_t v = add ? add[((size_t)l << a.log_n) + (g == 1 ? pos : auto_index(pos, g, a.log_n))] : 0;
            nttc::st_stream(out + t + 16 * k, sub_mul(ar, cv[k], x[k], w, v));
        }
    }
}

__device__ __forceinline__ uint64_t dec_value(const Ar<true> &ar, double x, uint64_t c0, uint64_t c1, const ModQ &)
{
    return ar.to_canon(ar.mul(x, Ar<true>::from_u64(c1)) + Ar<true>::from_u64(c0));
}
__device__ __forceinline__ uint64_t dec_value(const Ar<false> &ar, uint64_t x, uint64_t c0, uint64_t c1, const ModQ &m)
{
    return addmod(mulmod(ar.to_canon(x), c1, m), c0, m.q);
}
__device__ __forceinline__ uint64_t enc_value(const Ar<true> &ar, double e, double s, uint64_t a, uint64_t m,
                                              const ModQ &)
{
    return ar.to_canon(e + Ar<true>::from_u64(m) - ar.mul(s, Ar<true>::from_u64(a)));
}
__device__ __forceinline__ uint64_t enc_value(const Ar<false> &ar, uint64_t e, uint64_t s, uint64_t a, uint64_t m,
                                              const ModQ &md)
{
    return addmod(submod(ar.to_canon(e), mulmod(ar.to_canon(s), a, md), md.q), m, md.q);
}

// rows of s (and, ENC, of e after them) [1 or 2][limbs][N] after the column pass.  Every operand is read at the
// position the same thread writes, so pt may be c0's buffer, c0 m's and c1 a's.
template <bool F, bool ENC>
__global__ __launch_bounds__(128) void k_row_crypt(const uint64_t *__restrict__ rows, uint64_t *o0, uint64_t *o1,
                                                   const uint64_t *u, const uint64_t *v, uint32_t limbs,
                                                   uint32_t log_n, const ModQ *__restrict__ mods,
                                                   const void *__restrict__ tw_all)
{
    __shared__ E<F> lds[8 * 273];
    const uint32_t n1 = 1u << (log_n - 8), per = n1 / 8, sub = threadIdx.x >> 4, t = threadIdx.x & 15u;
    const uint32_t l = blockIdx.x / per, h = (blockIdx.x % per) * 8 + sub;
    const ModQ md = mods[l];
    const Ar<F> ar(md);
    const W<F> *tw = table<F>(tw_all, l, log_n);
    const size_t off = ((size_t)l << log_n) + (size_t)h * 256;
    E<F> x[kE], y[ENC ? kE : 1];
#pragma unroll
    for (int k = 0; k < kE; k++) x[k] = ar.from_raw(rows[off + t + 16 * k]);
    if constexpr (ENC) {
#pragma unroll
        for (int k = 0; k < kE; k++) y[k] = ar.from_raw(rows[((size_t)limbs << log_n) + off + t + 16 * k]);
    }
    uint64_t uv[kE], vv[kE];
#pragma unroll
    for (int k = 0; k < kE; k++) {
        uv[k] = u[off + t + 16 * k];
        vv[k] = v[off + t + 16 * k];
    }
    row_forward<F>(x, lds, tw, n1 + h, sub, t, ar);
    if constexpr (ENC) {
        row_forward<F>(y, lds, tw, n1 + h, sub, t, ar);
        // u = a, v = m
#pragma unroll
        for (int k = 0; k < kE; k++) {
            o0[off + t + 16 * k] = enc_value(ar, y[k], x[k], uv[k], vv[k], md);
            o1[off + t + 16 * k] = uv[k];
        }
    } else {
        // u = c0, v = c1
#pragma unroll
        for (int k = 0; k < kE; k++) o0[off + t + 16 * k] = dec_value(ar, x[k], uv[k], vv[k], md);
    }
}

// inverse row pass of one limb (index `limb`) of each polynomial c [polys][rows][N] into top [polys][N]
template <bool F>
__global__ __launch_bounds__(128) void k_top_row(uint64_t *top, const uint64_t *__restrict__ c, uint32_t rows,
                                                 uint32_t limb, uint32_t log_n, const ModQ *__restrict__ mods,
                                                 const void *__restrict__ itw)
{
    __shared__ E<F> lds[8 * 273];
    const uint32_t n1 = 1u << (log_n - 8), per = n1 / 8, sub = threadIdx.x >> 4, t = threadIdx.x & 15u;
    const uint32_t p = blockIdx.x / per, h = (blockIdx.x % per) * 8 + sub;
    const Ar<F> ar(mods[limb]);
    const W<F> *tw = table<F>(itw, limb, log_n);
    const uint64_t *in = c + (((size_t)p * rows + limb) << log_n) + (size_t)h * 256;
    uint64_t *out = top + ((size_t)p << log_n) + (size_t)h * 256;
    E<F> x[kE];
#pragma unroll
    for (int k = 0; k < kE; k++) x[k] = ar.from_u64(in[t + 16 * k]);
    nttc::transpose<8, true>(x, lds, sub, t);
    nttc::inv_low<8, F>(x, tw, n1 + h, t, ar);
    nttc::transpose<8, false>(x, lds, sub, t);
    nttc::inv_top<F>(x, tw, n1 + h, ar);
#pragma unroll
    for (int k = 0; k < kE; k++) out[t + 16 * k] = ar.to_raw(x[k]);
}

// its column pass, in place: centred coefficients as int64
template <int LOGS, bool F>
__global__ __launch_bounds__(256) void k_top_col(uint64_t *top, uint32_t limb, uint32_t log_n,
                                                 const ModQ *__restrict__ mods, const void *__restrict__ itw)
{
    constexpr uint32_t TS = (1u << LOGS) / 16, kCols = 4096u >> LOGS, kBpr = 256 / kCols;
    __shared__ E<F> lds[LOGS > 4 ? kCols * ((1u << LOGS) + (1u << LOGS) / 16 + 1) : 1];
    const Ar<F> ar(mods[limb]);
    const W<F> *tw = table<F>(itw, limb, log_n);
    const uint64_t q = mods[limb].q;
    const uint32_t col = threadIdx.x % kCols, t = threadIdx.x / kCols;
    uint64_t *base = top + ((size_t)(blockIdx.x / kBpr) << log_n) + (blockIdx.x % kBpr) * kCols + col;
    E<F> x[kE];
#pragma unroll
    for (int k = 0; k < kE; k++) x[k] = ar.from_raw(base[(size_t)(LOGS > 4 ? 16 * t + k : k) * 256]);
    if (LOGS > 4) {
        nttc::inv_low<LOGS, F>(x, tw, 1, t, ar);
        nttc::transpose<LOGS, false>(x, lds, col, t);
    }
    nttc::inv_top<F, true>(x, tw, 1, ar);
#pragma unroll
    for (int k = 0; k < kE; k++) {
        const uint64_t v = ar.to_canon(x[k]);
        base[(size_t)(t + TS * k) * 256] = v > (q >> 1) ? v - q : v;  // two's complement of the centred value
    }
}

template <bool F>
const void *fwd(const ckks_ctx *ctx)
{
    return F ? (const void *)ctx->d_twf : (const void *)ctx->d_tw;
}
template <bool F>
const void *inv(const ckks_ctx *ctx)
{
    return F ? (const void *)ctx->d_itwf : (const void *)ctx->d_itw;
}

template <bool F, int FIN>
void launch_fin(ckks_ctx *ctx, const FinArgs &a, const RotArgs &ra)
{
    const uint32_t n1 = 1u << (a.log_n - 8);
    const dim3 grid(a.polys * a.limbs * (n1 / 8)), block(128);
    if constexpr (!F) {
        if (a.polys % 8 == 0) {
            hipLaunchKernelGGL((k_row_fin<F, FIN, true>), grid, block, 0, ctx->stream, a, ra, ctx->d_mod, fwd<F>(ctx));
            return;
        }
    }
    hipLaunchKernelGGL((k_row_fin<F, FIN, false>), grid, block, 0, ctx->stream, a, ra, ctx->d_mod, fwd<F>(ctx));
}

// limb l of every polynomial as centred coefficients, int64 [polys][N]
template <bool F>
ckks_status top_coeffs(ckks_ctx *ctx, const uint64_t *c, uint32_t polys, uint32_t l, uint64_t *top)
{
    const uint32_t per = 1u << (ctx->log_n - 11);
    const double res = (double)polys * ctx->n, bf = F ? kOpsButterflyF64 : kOpsButterflyInt;
    prof_begin(ctx, K_NTT_INV_ROW, 16.0 * res, res * bf * 4);
    hipLaunchKernelGGL(k_top_row<F>, dim3(polys * per), dim3(128), 0, ctx->stream, top, c, l + 1, l, ctx->log_n,
                       ctx->d_mod, inv<F>(ctx));
    prof_end(ctx, K_NTT_INV_ROW);
    HIP_TRY(hipGetLastError());
    prof_begin(ctx, K_NTT_INV_COL, 16.0 * res, res * bf * (ctx->log_n - 8) / 2);
#define CK_COL(S)                                                                                                  \
    hipLaunchKernelGGL((k_top_col<S, F>), dim3(polys * (256 / (4096u >> S))), dim3(256), 0, ctx->stream, top, l,     \
                       ctx->log_n, ctx->d_mod, inv<F>(ctx))
    switch (ctx->log_n) {
    case 12: CK_COL(4); break;
    case 13: CK_COL(5); break;
    case 14: CK_COL(6); break;
    case 15: CK_COL(7); break;
    default: CK_COL(8); break;
    }
#undef CK_COL
    prof_end(ctx, K_NTT_INV_COL);
    HIP_TRY(hipGetLastError());
    return CKKS_OK;
}

// brackets a row pass over `rows` rows with its fused element-wise work, `words` words moved a position
void row_begin(ckks_ctx *ctx, bool f, double rows, double words)
{
    prof_begin(ctx, K_NTT_FWD_ROW, 8.0 * ctx->n * rows * words,
               rows * ctx->n * (f ? kOpsButterflyF64 : kOpsButterflyInt) * 4);
}

}  // namespace

bool fused_rows_ok(const ckks_ctx *ctx) { return ctx->log_n >= 12; }

ckks_status fused_rescale(ckks_ctx *ctx, const uint64_t *c, uint32_t polys, uint32_t l, uint64_t *out,
                          uint64_t *const *outs, uint64_t *work)
{
    RotArgs ra{};
    if (!out) {
        CK_REQUIRE(polys <= 2 * (uint32_t)kRotBatch, CKKS_EINVAL, "rescale of %u polynomials to separate outputs", polys);
        for (uint32_t r = 0; r < polys / 2; r++) ra.out[r] = outs[r];
    }
    uint64_t *top = work, *rows = top + (size_t)polys * ctx->n;
    // each transform in the arithmetic of its own primes
    if (ntt_map_f64(ctx, limb_range(l, 1)))
        CK_TRY(top_coeffs<true>(ctx, c, polys, l, top));
    else
        CK_TRY(top_coeffs<false>(ctx, c, polys, l, top));
    CK_TRY(launch_ntt_col_i64(ctx, (const int64_t *)top, rows, polys, l));
    FinArgs a{};
    a.in = rows;
    a.c = c;
    a.out = out;
    a.limbs = l;
    a.c_rows = l + 1;
    a.polys = polys;
    a.log_n = ctx->log_n;
    a.w = ctx->d_qlinv + (size_t)l * ctx->n_q;
    const bool f = ntt_uses_f64(ctx, l);
    row_begin(ctx, f, (double)polys * l, 3.0);
    if (f)
        launch_fin<true, FIN_RESCALE>(ctx, a, ra);
    else
        launch_fin<false, FIN_RESCALE>(ctx, a, ra);
    prof_end(ctx, K_NTT_FWD_ROW);
    HIP_TRY(hipGetLastError());
    return CKKS_OK;
}

ckks_status fused_moddown_int(ckks_ctx *ctx, uint32_t level, const RotArgs &ra, const uint64_t *u, const uint64_t *cw)
{
    FinArgs a{};
    a.in = cw;
    a.c = u;
    a.limbs = level + 1;
    a.c_rows = level + 1 + ctx->n_p;
    a.polys = 2 * ra.count;
    a.log_n = ctx->log_n;
    a.w = ctx->d_pinv;
    prof_begin(ctx, K_MODDOWN, 8.0 * ctx->n * a.limbs * ra.count * 7.0);
    launch_fin<false, FIN_MODDOWN>(ctx, a, ra);
    prof_end(ctx, K_MODDOWN);
    HIP_TRY(hipGetLastError());
    return CKKS_OK;
}

ckks_status fused_decrypt(ckks_ctx *ctx, uint64_t *pt, const uint64_t *c0, const uint64_t *c1, const int8_t *s,
                          uint32_t limbs, uint64_t *work)
{
    CK_TRY(launch_ntt_col_small(ctx, s, nullptr, work, limbs));
    const dim3 grid(limbs << (ctx->log_n - 11)), block(128);
    const bool f = ntt_uses_f64(ctx, limbs);
    row_begin(ctx, f, limbs, 4.0);
    if (f)
        hipLaunchKernelGGL((k_row_crypt<true, false>), grid, block, 0, ctx->stream, work, pt, (uint64_t *)nullptr, c0, c1,
                           limbs, ctx->log_n, ctx->d_mod, fwd<true>(ctx));
    else
        hipLaunchKernelGGL((k_row_crypt<false, false>), grid, block, 0, ctx->stream, work, pt, (uint64_t *)nullptr, c0,
                           c1, limbs, ctx->log_n, ctx->d_mod, fwd<false>(ctx));
    prof_end(ctx, K_NTT_FWD_ROW);
    HIP_TRY(hipGetLastError());
    return CKKS_OK;
}

ckks_status fused_encrypt(ckks_ctx *ctx, uint64_t *c0, uint64_t *c1, const uint64_t *a, const int8_t *s,
                          const int32_t *e, const uint64_t *m, uint32_t limbs, uint64_t *work)
{
    CK_TRY(launch_ntt_col_small(ctx, s, e, work, limbs));
    const dim3 grid(limbs << (ctx->log_n - 11)), block(128);
    const bool f = ntt_uses_f64(ctx, limbs);
    row_begin(ctx, f, 2.0 * limbs, 3.0);
    if (f)
        hipLaunchKernelGGL((k_row_crypt<true, true>), grid, block, 0, ctx->stream, work, c0, c1, a, m, limbs, ctx->log_n,
                           ctx->d_mod, fwd<true>(ctx));
    else
        hipLaunchKernelGGL((k_row_crypt<false, true>), grid, block, 0, ctx->stream, work, c0, c1, a, m, limbs, ctx->log_n,
                           ctx->d_mod, fwd<false>(ctx));
    prof_end(ctx, K_NTT_FWD_ROW);
    HIP_TRY(hipGetLastError());
    return CKKS_OK;
}
