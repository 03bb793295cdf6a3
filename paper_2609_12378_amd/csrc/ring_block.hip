// The small and medium rings with fp64 arithmetic (every prime below 2^50): steps that transform a row run as one launch
// with one block per row (ntt_block.h), the row's producer and consumer in the same kernel.  For N = 2^12 and 2^13 that
// is every step: a rotation is five launches (digits of c1; converted and transformed digits; key inner products;
// digits of their P rows; ModDown), a rescale two, an encryption or decryption one.  At these sizes a two-pass
// transform with an element-wise kernel on either side is bounded by its launches (about 4-5 us each, whatever the
// row count up to a few hundred); with many rows it moves each row through HBM four to six times.  At N = 2^14 it is the
// transforms, rescales and ModDowns of many rows (blk_rows, blk_rescales, blk_moddowns).
#include <algorithm>

#include "ckks_internal.h"
#include "ks_args.h"
#include "ntt_block.h"
#include "ops.h"

namespace {

using blk::A;
using nttc::GridSum;
using nttc::kE;
using nttc::ld_stream;
using nttc::st_stream;

// the ring constants a block needs for prime index p
struct Tab {
    const ModQ *mods;
    const double *twf, *itwf;
};
template <int LOGN>
__device__ __forceinline__ const double *table(const double *t, uint32_t prime)
{
    return t + ((size_t)prime << LOGN);
}
// ar with N^-1 f mod q (f canonical) as its inverse-transform factor
__device__ __forceinline__ A scaled(const A &ar, double f)
{
    A s = ar;
    s.ninv = ar.scaled_twiddle(f);
    return s;
}

// Words a kernel combines with the transformed row, at the thread's row positions.  EARLY: loaded before the
// transform, so that they arrive during it, and the conversion keeps twice as many loads in flight: up to 236
// registers a thread, right while the grid leaves a CU no second block anyway (early_loads).  Else they are loaded
// where they are used, in 128 registers, so that other blocks hide the wait.
template <int LOGN, bool EARLY>
struct Words {
    static constexpr bool kEarly = EARLY;
    uint64_t v[kEarly ? kE : 1];
    const uint64_t *p;
    __device__ explicit Words(const uint64_t *row) : p(row)
    {
        if constexpr (kEarly) {
#pragma unroll
            for (int k = 0; k < kE; k++) v[k] = row[blk::row_pos(threadIdx.x, k)];
        }
    }
    __device__ uint64_t get(int k) const
    {
        if constexpr (kEarly) return v[k];
        return p[blk::row_pos(threadIdx.x, k)];
    }
};

// the same for an addend read through the automorphism g (1: none); row null: no addend
template <int LOGN, bool EARLY>
struct Addend {
    static constexpr bool kEarly = EARLY;
    uint64_t v[kEarly ? kE : 1];
    const uint64_t *p;
    uint32_t g;
    __device__ Addend(const uint64_t *row, uint32_t g_) : p(row), g(g_)
    {
        if constexpr (kEarly) {
            if (p) {
#pragma unroll
                for (int k = 0; k < kE; k++) v[k] = p[at(k)];
            } else {
#pragma unroll
                for (int k = 0; k < kE; k++) v[k] = 0;
            }
        }
    }
    __device__ uint32_t at(int k) const
    {
        const uint32_t q = blk::row_pos(threadIdx.x, k);
        return g == 1 ? q : auto_index(q, g, LOGN);
    }
    __device__ uint64_t get(int k) const
    {
        if constexpr (kEarly) return v[k];
        return p ? p[at(k)] : 0;
    }
};

// ---- plain transforms: row r of the launch is group r / map.n, limb r % map.n -------------------------------------
template <int LOGN, bool INV>
__global__ __launch_bounds__(blk::Shape<LOGN>::NT) void k_blk_ntt(uint64_t *dst, uint32_t dst_stride,
                                                                  const uint64_t *src, uint32_t src_stride,
                                                                  LimbMap map, Tab tb)
{
    __shared__ double lds[blk::Shape<LOGN>::kLds];
    const uint32_t b = blockIdx.x / map.n, limb = blockIdx.x % map.n, prime = map.prime[limb], t = threadIdx.x;
    const A ar(tb.mods[prime]);
    const double *tw = table<LOGN>(INV ? tb.itwf : tb.twf, prime);
    const blk::ColTw<LOGN> cw(tw);
    const blk::RowTw<LOGN> rw(tw);
    const uint64_t *in = src + (((size_t)b * src_stride + limb) << LOGN);
    uint64_t *out = dst + (((size_t)b * dst_stride + limb) << LOGN);
    double x[kE];
#pragma unroll
    for (int k = 0; k < kE; k++) x[k] = A::from_u64(ld_stream(in + (INV ? blk::row_pos(t, k) : blk::col_pos<LOGN>(t, k))));
    if (INV)
        blk::inverse<LOGN>(x, lds, cw, rw, ar, ar);
    else
        blk::forward<LOGN>(x, lds, cw, rw, ar);
#pragma unroll
    for (int k = 0; k < kE; k++)
        st_stream(out + (INV ? blk::col_pos<LOGN>(t, k) : blk::row_pos(t, k)), ar.to_canon(x[k]));
}

// forward transform of signed coefficients m[b] modulo q_l into out[b][l]
template <int LOGN>
__global__ __launch_bounds__(blk::Shape<LOGN>::NT) void k_blk_from_i64(const int64_t *__restrict__ m, uint64_t *out,
                                                                       uint32_t limbs, Tab tb)
{
    __shared__ double lds[blk::Shape<LOGN>::kLds];
    const uint32_t l = blockIdx.x % limbs, b = blockIdx.x / limbs, t = threadIdx.x;
    const ModQ md = tb.mods[l];
    const A ar(md);
    const blk::ColTw<LOGN> cw(table<LOGN>(tb.twf, l));
    const blk::RowTw<LOGN> rw(table<LOGN>(tb.twf, l));
    const int64_t *in = m + ((size_t)b << LOGN);
    double x[kE];
    bool big = false;
#pragma unroll
    for (int k = 0; k < kE; k++) {
        const int64_t v = in[blk::col_pos<LOGN>(t, k)];
        big |= v > (1ll << 52) || v < -(1ll << 52);
        x[k] = ar.red((double)v);
    }
    if (__any(big)) {
        // rare: the general reduction, one copy of it in a loop (a register chosen by comparison)
#pragma unroll 1
        for (int k = 0; k < kE; k++) {
            const double xk = ar.from_i64(in[blk::col_pos<LOGN>(t, k)], md);
#pragma unroll
            for (int i = 0; i < kE; i++) x[i] = i == k ? xk : x[i];
        }
    }
    blk::forward<LOGN>(x, lds, cw, rw, ar);
    uint64_t *o = out + ((size_t)blockIdx.x << LOGN);
#pragma unroll
    for (int k = 0; k < kE; k++) st_stream(o + blk::row_pos(t, k), ar.to_canon(x[k]));
}

// ---- encryption and decryption: one block per limb ----------------------------------------------------------------
// c0 = NTT(e) + m - a NTT(s), c1 = a.  m and a are read at the positions the same thread writes, so c0 may be m's
// buffer and c1 a's.  Sums below 4.1 + 1 + 2.1 q.
template <int LOGN>
__global__ __launch_bounds__(blk::Shape<LOGN>::NT) void k_blk_encrypt(uint64_t *c0, uint64_t *c1, const uint64_t *a,
                                                                      const int8_t *__restrict__ s,
                                                                      const int32_t *__restrict__ e,
                                                                      const uint64_t *m, Tab tb)
{
    __shared__ double lds[blk::Shape<LOGN>::kLds];
    const uint32_t l = blockIdx.x, t = threadIdx.x;
    const A ar(tb.mods[l]);
    const double *tw = table<LOGN>(tb.twf, l);
    const blk::ColTw<LOGN> cw(tw);
    const size_t row = (size_t)l << LOGN;
    const Words<LOGN, true> aw(a + row);
    double x[kE], p[kE];
#pragma unroll
    for (int k = 0; k < kE; k++) x[k] = (double)s[blk::col_pos<LOGN>(t, k)];
    {
        const blk::RowTw<LOGN> rw(tw);
        blk::forward<LOGN>(x, lds, cw, rw, ar);
    }
    // the row's twiddles again (an opaque copy of the pointer: not held in registers in between)
    asm volatile("" : "+s"(tw));
#pragma unroll
    for (int k = 0; k < kE; k++) p[k] = ar.mul(x[k], A::from_u64(aw.get(k)));
#pragma unroll
    for (int k = 0; k < kE; k++) x[k] = (double)e[blk::col_pos<LOGN>(t, k)];
    const Words<LOGN, true> mw(m + row);
    __syncthreads();
    {
        const blk::RowTw<LOGN> rw(tw);
        blk::forward<LOGN>(x, lds, cw, rw, ar);
    }
#pragma unroll
    for (int k = 0; k < kE; k++) {
        const size_t i = row + blk::row_pos(t, k);
        const double v = x[k] + A::from_u64(mw.get(k)) - p[k];
        c0[i] = ar.to_canon(v);
        c1[i] = aw.get(k);
    }
}

// pt = c0 + c1 NTT(s)
template <int LOGN>
__global__ __launch_bounds__(blk::Shape<LOGN>::NT) void k_blk_decrypt(uint64_t *pt, const uint64_t *c0,
                                                                      const uint64_t *c1,
                                                                      const int8_t *__restrict__ s, Tab tb)
{
    __shared__ double lds[blk::Shape<LOGN>::kLds];
    const uint32_t l = blockIdx.x, t = threadIdx.x;
    const A ar(tb.mods[l]);
    const blk::ColTw<LOGN> cw(table<LOGN>(tb.twf, l));
    const blk::RowTw<LOGN> rw(table<LOGN>(tb.twf, l));
    const size_t row = (size_t)l << LOGN;
    const Words<LOGN, true> w0(c0 + row), w1(c1 + row);
    double x[kE];
#pragma unroll
    for (int k = 0; k < kE; k++) x[k] = (double)s[blk::col_pos<LOGN>(t, k)];
    blk::forward<LOGN>(x, lds, cw, rw, ar);
#pragma unroll
    for (int k = 0; k < kE; k++)
        pt[row + blk::row_pos(t, k)] = ar.to_canon(ar.mul(x[k], A::from_u64(w1.get(k))) + A::from_u64(w0.get(k)));
}

// ---- rescale ------------------------------------------------------------------------------------------------------
// the top limb of polynomial p (c: [polys][l + 1][N]) as centred coefficients, integer-valued doubles
template <int LOGN>
__global__ __launch_bounds__(blk::Shape<LOGN>::NT) void k_blk_rescale_top(double *top, const uint64_t *__restrict__ c,
                                                                          uint32_t l, Tab tb)
{
    __shared__ double lds[blk::Shape<LOGN>::kLds];
    const uint32_t t = threadIdx.x;
    const A ar(tb.mods[l]);
    const blk::ColTw<LOGN> cw(table<LOGN>(tb.itwf, l));
    const blk::RowTw<LOGN> rw(table<LOGN>(tb.itwf, l));
    const uint64_t *in = c + (((size_t)blockIdx.x * (l + 1) + l) << LOGN);
    double x[kE];
#pragma unroll
    for (int k = 0; k < kE; k++) x[k] = A::from_u64(in[blk::row_pos(t, k)]);
    blk::inverse<LOGN>(x, lds, cw, rw, ar, ar);
    double *o = top + ((size_t)blockIdx.x << LOGN);
#pragma unroll
    for (int k = 0; k < kE; k++) o[blk::col_pos<LOGN>(t, k)] = ar.red(x[k]);
}
// out_i = (c_i - NTT(top mod q_i)) q_l^-1
template <int LOGN, bool EARLY>
__global__ __launch_bounds__(blk::Shape<LOGN>::NT, EARLY ? 1 : 4)
void k_blk_rescale(uint64_t *out, const uint64_t *__restrict__ c, const double *__restrict__ top, uint32_t l,
                   const ulonglong2 *__restrict__ qlinv, Tab tb)
{
    __shared__ double lds[blk::Shape<LOGN>::kLds];
    const uint32_t i = blockIdx.x % l, poly = blockIdx.x / l, t = threadIdx.x;
    const A ar(tb.mods[i]);
    const blk::ColTw<LOGN> cw(table<LOGN>(tb.twf, i));
    const blk::RowTw<LOGN> rw(table<LOGN>(tb.twf, i));
    const double *tp = top + ((size_t)poly << LOGN);
    double x[kE];
#pragma unroll
    for (int k = 0; k < kE; k++) x[k] = ar.red(tp[blk::col_pos<LOGN>(t, k)]);
    const Words<LOGN, EARLY> cv(c + (((size_t)poly * (l + 1) + i) << LOGN));
    blk::forward<LOGN>(x, lds, cw, rw, ar);
    uint64_t *o = out + ((size_t)blockIdx.x << LOGN);
    const double w = (double)qlinv[i].x;
#pragma unroll
    for (int k = 0; k < kE; k++) {
        const uint32_t p = blk::row_pos(t, k);
        st_stream(o + p, ar.to_canon(ar.mul(A::from_u64(cv.get(k)) - x[k], w)));
    }
}

// ---- key switching ------------------------------------------------------------------------------------------------
// The conversion constants of a ModUp's digits at one level (fp64 tables of ConvDev)
struct Digits {
    uint32_t nd, alpha, L, K, n_q;
    const double *inv[kMaxPrimes], *mod[kMaxPrimes];
};
// A polynomial that is switched: c1 at base + r stride for entry r of the batch, or (b set) the product of the second
// components of the ciphertexts a and b ([2][L][N] each), formed where it is read
struct Source {
    const uint64_t *base;
    size_t stride;
    const uint64_t *b;
};

// acc[k] += y_i w_i for G consecutive sources, all their loads issued first
template <int LOGN, int G, int W>
__device__ __forceinline__ void convert_group(GridSum (&acc)[W], const double *__restrict__ y, int i, int k0,
                                              const double *__restrict__ w, int wstride)
{
    double v[G][W];
#pragma unroll
    for (int j = 0; j < G; j++)
#pragma unroll
        for (int k = 0; k < W; k++) v[j][k] = y[((size_t)(i + j) << LOGN) + blk::col_pos<LOGN>(threadIdx.x, k0 + k)];
#pragma unroll
    for (int j = 0; j < G; j++) {
        const double wi = w[(i + j) * wstride];
#pragma unroll
        for (int k = 0; k < W; k++) acc[k].add(v[j][k], wi);
    }
}

// sum_i y_i w_i for 16 points of the column layout (y: ns rows of centred digits), |x| <= q/2
template <int LOGN, bool EARLY>
__device__ __forceinline__ void convert(double (&x)[kE], const double *__restrict__ y, int ns,
                                        const double *__restrict__ w, int wstride, const A &ar)
{
    // eight points at a time (sixteen of the two-word sums and the loads in flight would not fit 128 registers), or
    // all sixteen, half as many waits on memory
    constexpr int W = EARLY ? 16 : 8, G = EARLY ? 4 : 3;
#pragma unroll
    for (int k0 = 0; k0 < kE; k0 += W) {
        GridSum acc[W];
        for (int i0 = 0; i0 < ns; i0 += GridSum::kTerms) {
            if (i0) {
#pragma unroll
                for (int k = 0; k < W; k++) acc[k].fold(ar);
            }
            const int i1 = min(ns, i0 + GridSum::kTerms);
            int i = i0;
#pragma unroll 1
            for (; i + G <= i1; i += G) convert_group<LOGN, G>(acc, y, i, k0, w, wstride);
            if (G == 4 && i + 3 <= i1) {
                convert_group<LOGN, 3>(acc, y, i, k0, w, wstride);
                i += 3;
            }
            if (i + 2 <= i1) {
                convert_group<LOGN, 2>(acc, y, i, k0, w, wstride);
                i += 2;
            }
            if (i < i1) convert_group<LOGN, 1>(acc, y, i, k0, w, wstride);
        }
#pragma unroll
        for (int k = 0; k < W; k++) x[k0 + k] = ar.red(acc[k].value(ar));
    }
}

// y[r][l] = the centred conversion digit [c1_l Qhat_l^-1] of limb l (its digit's constant folded into the inverse
// transform's last stage), as doubles; grid (L, count)
template <int LOGN, bool TENSOR>
__global__ __launch_bounds__(blk::Shape<LOGN>::NT) void k_blk_digits(double *y, Source src, Digits dg, Tab tb)
{
    __shared__ double lds[blk::Shape<LOGN>::kLds];
    const uint32_t l = blockIdx.x, r = blockIdx.y, t = threadIdx.x, j = l / dg.alpha;
    const A ar(tb.mods[l]);
    const blk::ColTw<LOGN> cw(table<LOGN>(tb.itwf, l));
    const blk::RowTw<LOGN> rw(table<LOGN>(tb.itwf, l));
    const uint64_t *in = src.base + r * src.stride + ((size_t)l << LOGN);
    double x[kE];
#pragma unroll
    for (int k = 0; k < kE; k++) {
        const uint32_t p = blk::row_pos(t, k);
        x[k] = A::from_u64(in[p]);
        if (TENSOR) x[k] = ar.mul(x[k], A::from_u64(src.b[((size_t)(dg.L + l) << LOGN) + p]));
    }
    blk::inverse<LOGN>(x, lds, cw, rw, ar, scaled(ar, dg.inv[j][l - j * dg.alpha]));
    double *o = y + (((size_t)r * dg.L + l) << LOGN);
#pragma unroll
    for (int k = 0; k < kE; k++) o[blk::col_pos<LOGN>(t, k)] = ar.red(x[k]);
}

// row `row` of digit j of entry r: the conversion of the digit's limbs transformed, or for the digit's own limbs the
// polynomial itself; grid (ext, nd, count)
template <int LOGN, bool TENSOR, bool EARLY>
__global__ __launch_bounds__(blk::Shape<LOGN>::NT, EARLY ? 1 : 4)
void k_blk_modup(uint64_t *digits, const double *__restrict__ y, Source src, Digits dg, Tab tb)
{
    __shared__ double lds[blk::Shape<LOGN>::kLds];
    const uint32_t row = blockIdx.x, j = blockIdx.y, r = blockIdx.z, t = threadIdx.x, ext = dg.L + dg.K;
    const uint32_t lo = j * dg.alpha, hi = min(lo + dg.alpha, dg.L);
    const uint32_t prime = row < dg.L ? row : dg.n_q + (row - dg.L);
    const A ar(tb.mods[prime]);
    uint64_t *o = digits + ((((size_t)r * dg.nd + j) * ext + row) << LOGN);
    if (row >= lo && row < hi) {
        const uint64_t *in = src.base + r * src.stride + ((size_t)row << LOGN);
#pragma unroll
        for (int k = 0; k < kE; k++) {
            const uint32_t p = blk::row_pos(t, k);
            uint64_t v = in[p];
            if (TENSOR)
                v = ar.to_canon(ar.mul(A::from_u64(v), A::from_u64(src.b[((size_t)(dg.L + row) << LOGN) + p])));
            o[p] = v;
        }
        return;
    }
    const uint32_t target = row < lo ? row : row - (hi - lo);
    double x[kE];
    convert<LOGN, EARLY>(x, y + (((size_t)r * dg.L + lo) << LOGN), (int)(hi - lo), dg.mod[j] + target,
                  (int)(ext - (hi - lo)), ar);
    const blk::ColTw<LOGN> cw(table<LOGN>(tb.twf, prime));
    const blk::RowTw<LOGN> rw(table<LOGN>(tb.twf, prime));
    blk::forward<LOGN>(x, lds, cw, rw, ar);
#pragma unroll
    for (int k = 0; k < kE; k++) o[blk::row_pos(t, k)] = ar.to_canon(x[k]);
}

// u[r][k][row] = sum_j sigma_{g_r}(d_j)[row] key_{r,j}[k][prime(row)] over Q_level u P (u: [count][2][ext][N],
// canonical).  Element-wise and apart from the transforms on either side: it reads 24 nd bytes a position, for which
// one position a thread with every load issued before the first product keeps more of them in flight over more of
// the chip than the blocks of a few rows would.  Products below 0.875 q, the sum range-reduced every four digits.
// ND > 0: the digit count at compile time.
template <int ND>
__global__ __launch_bounds__(256) void k_blk_key(uint64_t *u, RotArgs ra, uint32_t nd, uint32_t L, uint32_t K,
                                                 uint32_t n_q, const ModQ *__restrict__ mods, uint32_t log_n)
{
    const uint32_t pos = blockIdx.x * 256 + threadIdx.x, row = blockIdx.y, r = blockIdx.z;
    const uint32_t ext = L + K, rows = n_q + K, prime = row < L ? row : n_q + (row - L);
    const uint32_t sc = auto_index(pos, ra.g[r], log_n);
    const uint64_t *dig = ra.dig[r] + ((size_t)row << log_n) + sc;
    const uint64_t *key = ra.key[r] + ((size_t)prime << log_n) + pos;
    const size_t dstride = (size_t)ext << log_n, kstride = (size_t)rows << log_n;
    const A ar(mods[prime]);
    double u0 = 0.0, u1 = 0.0;
    if constexpr (ND > 0) {
        uint64_t dv[ND], bv[ND], av[ND];
#pragma unroll
        for (int j = 0; j < ND; j++) {
            dv[j] = dig[j * dstride];
            bv[j] = ld_stream(key + 2 * j * kstride);
            av[j] = ld_stream(key + (2 * j + 1) * kstride);
        }
#pragma unroll
        for (int j = 0; j < ND; j++) {
            u0 += ar.mul(A::from_u64(dv[j]), A::from_u64(bv[j]));
            u1 += ar.mul(A::from_u64(dv[j]), A::from_u64(av[j]));
        }
    } else {
        for (uint32_t j = 0; j < nd; j++) {
            const double d = A::from_u64(dig[j * dstride]);
            u0 += ar.mul(d, A::from_u64(ld_stream(key + 2 * j * kstride)));
            u1 += ar.mul(d, A::from_u64(ld_stream(key + (2 * j + 1) * kstride)));
            if ((j & 3) == 3) {
                u0 = ar.red(u0);
                u1 = ar.red(u1);
            }
        }
    }
    uint64_t *o = u + (((size_t)r * 2 * ext + row) << log_n) + pos;
    o[0] = ar.to_canon(u0);
    o[dstride] = ar.to_canon(u1);
}

// ModDown of polynomials u ([polys][L + K][N]), step 1: P row i of each to its centred conversion digit, in place
// (a thread's words are in registers before the first block barrier and written after the last); grid (K, polys)
template <int LOGN>
__global__ __launch_bounds__(blk::Shape<LOGN>::NT) void k_blk_moddown_p(uint64_t *u, uint32_t L, uint32_t K,
                                                                        uint32_t n_q,
                                                                        const double *__restrict__ pinv_digit, Tab tb)
{
    __shared__ double lds[blk::Shape<LOGN>::kLds];
    const uint32_t i = blockIdx.x, t = threadIdx.x, prime = n_q + i;
    const A ar(tb.mods[prime]);
    uint64_t *row = u + (((size_t)blockIdx.y * (L + K) + L + i) << LOGN);
    const blk::ColTw<LOGN> cw(table<LOGN>(tb.itwf, prime));
    const blk::RowTw<LOGN> rw(table<LOGN>(tb.itwf, prime));
    double x[kE];
#pragma unroll
    for (int k = 0; k < kE; k++) x[k] = A::from_u64(row[blk::row_pos(t, k)]);
    blk::inverse<LOGN>(x, lds, cw, rw, ar, scaled(ar, pinv_digit[i]));
#pragma unroll
    for (int k = 0; k < kE; k++) row[blk::col_pos<LOGN>(t, k)] = A::to_raw(ar.red(x[k]));
}

// step 2: out_k[i] = (u_k[i] - NTT(Conv)[i]) P^-1 + add_k[i], add_k read through the automorphism g (1: none).
// Magnitudes (units of q): u 1, transform 4.1, P^-1 product 2.5, addend 1 (tensor: 1.8).
enum { ADD_ROWS = 0, ADD_TENSOR = 1 };
template <int LOGN, int MODE, bool EARLY>
__device__ __forceinline__ void moddown_finish(double *lds, uint64_t *o, const uint64_t *up, uint32_t i, uint32_t k,
                                               const uint64_t *add, uint32_t g, const uint64_t *ta,
                                               const uint64_t *tb2, uint32_t L, uint32_t K, const double *pmod,
                                               const ulonglong2 *pinv, const Tab &tb)
{
    const uint32_t t = threadIdx.x;
    const A ar(tb.mods[i]);
    const size_t row = (size_t)i << LOGN;
    double x[kE];
    convert<LOGN, EARLY>(x, (const double *)up + ((size_t)L << LOGN), (int)K, pmod + i, (int)L, ar);
    const blk::ColTw<LOGN> cw(table<LOGN>(tb.twf, i));
    const blk::RowTw<LOGN> rw(table<LOGN>(tb.twf, i));
    const Words<LOGN, EARLY> uw(up + row);
    const Addend<LOGN, EARLY> aw(MODE == ADD_ROWS && add ? add + row : nullptr, g);
    blk::forward<LOGN>(x, lds, cw, rw, ar);
    const double pi = (double)pinv[i].x;
#pragma unroll
    for (int e = 0; e < kE; e++) {
        const uint32_t p = blk::row_pos(t, e);
        double v = ar.mul(A::from_u64(uw.get(e)) - x[e], pi);
        if (MODE == ADD_TENSOR) {
            const size_t q0 = row + p, q1 = q0 + ((size_t)L << LOGN);
            if (k == 0)
                v += ar.mul(A::from_u64(ta[q0]), A::from_u64(tb2[q0]));
            else
                v += ar.mul(A::from_u64(ta[q0]), A::from_u64(tb2[q1])) +
                     ar.mul(A::from_u64(ta[q1]), A::from_u64(tb2[q0]));
        } else {
            v += A::from_u64(aw.get(e));
        }
        st_stream(o + p, ar.to_canon(v));
    }
}
// polynomial k of `polys` (grid (L, polys)): add0 for the first, add1 for the second
template <int LOGN, bool EARLY>
__global__ __launch_bounds__(blk::Shape<LOGN>::NT, EARLY ? 1 : 4) void k_blk_moddown(uint64_t *out, const uint64_t *u,
                                                                      const uint64_t *add0, uint32_t add0_g,
                                                                      const uint64_t *add1, uint32_t L, uint32_t K,
                                                                      const double *__restrict__ pmod,
                                                                      const ulonglong2 *__restrict__ pinv, Tab tb)
{
    __shared__ double lds[blk::Shape<LOGN>::kLds];
    const uint32_t i = blockIdx.x, k = blockIdx.y;
    moddown_finish<LOGN, ADD_ROWS, EARLY>(lds, out + (((size_t)k * L + i) << LOGN), u + ((size_t)k * (L + K) << LOGN),
                                          i, k, k == 0 ? add0 : k == 1 ? add1 : nullptr, k == 0 ? add0_g : 1u, nullptr,
                                          nullptr, L, K, pmod, pinv, tb);
}
// component k of rotation r (grid (L, 2, count)): sigma_g(c0) for the first, add1 (if set) for the second; with
// ADD_TENSOR the first two components of the tensor product of ta and tb2
template <int LOGN, int MODE, bool EARLY>
__global__ __launch_bounds__(blk::Shape<LOGN>::NT, EARLY ? 1 : 4)
void k_blk_finish(RotArgs ra, const uint64_t *u, uint32_t L, uint32_t K, const double *__restrict__ pmod,
                  const ulonglong2 *__restrict__ pinv, const uint64_t *ta, const uint64_t *tb2, Tab tb)
{
    __shared__ double lds[blk::Shape<LOGN>::kLds];
    const uint32_t i = blockIdx.x, k = blockIdx.y, r = blockIdx.z;
    moddown_finish<LOGN, MODE, EARLY>(lds, ra.out[r] + (((size_t)k * L + i) << LOGN),
                               u + (((size_t)r * 2 + k) * (L + K) << LOGN), i, k, k ? ra.add1[r] : ra.c0[r],
                               k ? 1u : ra.g[r], ta, tb2, L, K, pmod, pinv, tb);
}

Tab tab_of(const ckks_ctx *ctx) { return Tab{ctx->d_mod, ctx->d_twf, ctx->d_itwf}; }

// one launch for the context's ring degree; CK_BLK13: of the steps that N = 2^14 does not take
#define CK_BLK13(KERNEL, GRID, ...)                                                                                \
    do {                                                                                                           \
        if (ctx->log_n == 12)                                                                                      \
            hipLaunchKernelGGL((KERNEL(12)), GRID, dim3(blk::Shape<12>::NT), 0, ctx->stream, __VA_ARGS__);           \
        else                                                                                                       \
            hipLaunchKernelGGL((KERNEL(13)), GRID, dim3(blk::Shape<13>::NT), 0, ctx->stream, __VA_ARGS__);           \
    } while (0)
#define CK_BLK(KERNEL, GRID, ...)                                                                                  \
    do {                                                                                                           \
        switch (ctx->log_n) {                                                                                      \
        case 12: hipLaunchKernelGGL((KERNEL(12)), GRID, dim3(blk::Shape<12>::NT), 0, ctx->stream, __VA_ARGS__); break; \
        case 13: hipLaunchKernelGGL((KERNEL(13)), GRID, dim3(blk::Shape<13>::NT), 0, ctx->stream, __VA_ARGS__); break; \
        default: hipLaunchKernelGGL((KERNEL(14)), GRID, dim3(blk::Shape<14>::NT), 0, ctx->stream, __VA_ARGS__); break; \
        }                                                                                                          \
    } while (0)

// K_E(LG) where a grid of `blocks` takes the early loads (N = 2^14, 1024 threads: never more than 128 registers),
// else K_L(LG)
bool early_loads(const ckks_ctx *ctx, size_t blocks) { return ctx->log_n <= 13 && blocks <= 256; }
#define CK_BLK_E(BLOCKS, GRID, ...)                                                                                \
    do {                                                                                                           \
        if (early_loads(ctx, BLOCKS))                                                                              \
            CK_BLK(CK_E, GRID, __VA_ARGS__);                                                                       \
        else                                                                                                       \
            CK_BLK(CK_L, GRID, __VA_ARGS__);                                                                       \
    } while (0)
#define CK_BLK13_E(BLOCKS, GRID, ...)                                                                              \
    do {                                                                                                           \
        if (early_loads(ctx, BLOCKS))                                                                              \
            CK_BLK13(CK_E, GRID, __VA_ARGS__);                                                                     \
        else                                                                                                       \
            CK_BLK13(CK_L, GRID, __VA_ARGS__);                                                                     \
    } while (0)

ckks_status launch_moddown_p(ckks_ctx *ctx, uint64_t *u, uint32_t polys, uint32_t L, uint32_t K, const ConvDev *cd)
{
    prof_begin(ctx, K_NTT_INV_ROW, 16.0 * polys * K * ctx->n);
#define CK_K(LG) k_blk_moddown_p<LG>
    CK_BLK(CK_K, dim3(K, polys), u, L, K, ctx->n_q, cd->d_qhat_inv_f, tab_of(ctx));
#undef CK_K
    prof_end(ctx, K_NTT_INV_ROW);
    HIP_TRY(hipGetLastError());
    return CKKS_OK;
}

// the key inner products of a batch over every row: u [count][2][level + 1 + n_p][N]
ckks_status blk_key_product(ckks_ctx *ctx, uint32_t level, const RotArgs &ra, uint64_t *u)
{
    const uint32_t L = level + 1, K = ctx->n_p, nd = n_digits(ctx, level);
    const dim3 grid(ctx->n / 256, L + K, ra.count), block(256);
    prof_begin(ctx, K_KEYIP, 8.0 * ctx->n * (L + K) * (ra.count * (2.0 * nd + 2.0) + nd));
#define CK_KEY(ND)                                                                                                 \
    hipLaunchKernelGGL(k_blk_key<ND>, grid, block, 0, ctx->stream, u, ra, nd, L, K, ctx->n_q, ctx->d_mod, ctx->log_n)
    switch (nd) {
    case 1: CK_KEY(1); break;
    case 2: CK_KEY(2); break;
    case 3: CK_KEY(3); break;
    case 4: CK_KEY(4); break;
    default: CK_KEY(0); break;
    }
#undef CK_KEY
    prof_end(ctx, K_KEYIP);
    HIP_TRY(hipGetLastError());
    return CKKS_OK;
}

}  // namespace

// N = 2^14: a block is 1024 threads and all of a CU's LDS, 15 us a row with nothing to hide its waits, so the two
// passes (about 6 us each while they leave the chip idle) are faster for a few rows: up to 128, whose column pass is 512
// blocks, two a CU.  A forward and an inverse transform as a program calls them: 64 rows 33.8 us here against 26.7, 96
// rows 34.2 against 30.7, 128 rows 34.6 against 33.4, 129 rows 34.7 against 39.6, 160 rows 35.0 against 41.5, 186 rows
// 36.9 against 47.2, in whatever groups the rows come
bool blk_rows(const ckks_ctx *ctx, size_t rows) { return blk_ring(ctx) && (ctx->log_n < 14 || rows > 128); }

// the same for a rescale, two launches here and four there, by the rows out: 96 rows 32.4 against 29.7 us, 128 rows 35.3
// against 34.1 in the kernels alone, 160 rows 34.7 against 36.3, 186 rows 37.3 against 41.1 in the kernels, 384 rows 53
// against 59
bool blk_rescales(const ckks_ctx *ctx, size_t rows) { return blk_rows(ctx, rows); }

// the same for the first pass from coefficients, which at N = 2^14 has one plaintext's limbs (64 rows 15.4 against 15.0)
bool blk_from_i64(const ckks_ctx *ctx) { return blk_ring(ctx) && ctx->log_n < 14; }

// the same for one encryption and decryption (fused_row.hip: two launches)
bool blk_crypt(const ckks_ctx *ctx, uint32_t limbs)
{
    return blk_ring(ctx) && ntt_uses_f64(ctx, limbs) && ctx->log_n < 14;
}

// the same for a ModDown of `polys` polynomials, by the rows it transforms back.  Whole rows less two passes, in the time
// of a projection that ends in one: 24 rows +5 to +14 us (of 330 to 490), 48 rows +9 (24 limbs), 0 (12 and 6 limbs) and
// -3 (3 limbs), 72 rows -4 to -5, 90 rows -11, 96 to 288 rows -1 to -21
bool blk_moddowns(const ckks_ctx *ctx, uint32_t level, uint32_t polys)
{
    return blk_ring(ctx) && f64_switch(ctx, level) && (ctx->log_n < 14 || (size_t)polys * (level + 1) > 48);
}

bool blk_ring(const ckks_ctx *ctx) { return ctx->log_n >= blk::kMinLog && ctx->log_n <= blk::kMaxLog && !ctx->int_only; }

// A ModUp and a batch of rotations: not at N = 2^14, where the two-pass kernels (modup.hip, keyswitch.hip) keep the q
// rows of the key products on chip and their grids are not bound to whole rows.  24 + 8 limbs, 1, 9 and 32 rotations of
// 24 limbs 100, 201 and 585 us with the whole-row ModDown against 76, 192 and 465 in two passes, of 8 limbs 85, 117 and
// 266 against 52, 86 and 184; 12 + 4 limbs, 9 rotations of 8 limbs 96 against 85.  The exception is 32 rotations of 1 to
// 4 limbs under at most 4 special primes: kernels of 81 to 100 us there and 73 to 101 here, but a call bound by its
// caller's side, for which two launches fewer were 98 us against 104
bool blk_switch(const ckks_ctx *ctx, uint32_t level)
{
    return blk_ring(ctx) && ctx->log_n < 14 && f64_switch(ctx, level);
}

ckks_status blk_ntt(ckks_ctx *ctx, uint64_t *dst, uint32_t dst_stride, const uint64_t *src, uint32_t src_stride,
                    uint32_t batch, const LimbMap &map, bool inverse)
{
    const dim3 grid(batch * map.n);
    const Tab tb = tab_of(ctx);
    const double res = (double)batch * map.n * ctx->n;
    const KClass kc = inverse ? K_NTT_INV_ROW : K_NTT_FWD_ROW;
    prof_begin(ctx, kc, 16.0 * res, res * kOpsButterflyF64 * ctx->log_n / 2);
#define CK_K(LG) k_blk_ntt<LG, true>
    if (inverse) CK_BLK(CK_K, grid, dst, dst_stride, src, src_stride, map, tb);
#undef CK_K
#define CK_K(LG) k_blk_ntt<LG, false>
    if (!inverse) CK_BLK(CK_K, grid, dst, dst_stride, src, src_stride, map, tb);
#undef CK_K
    prof_end(ctx, kc);
    HIP_TRY(hipGetLastError());
    return CKKS_OK;
}

ckks_status blk_ntt_from_i64(ckks_ctx *ctx, const int64_t *m, uint64_t *out, uint32_t batch, uint32_t limbs)
{
    const double res = (double)batch * limbs * ctx->n;
    prof_begin(ctx, K_NTT_FWD_ROW, 8.0 * batch * ctx->n * (1 + limbs), res * kOpsButterflyF64 * ctx->log_n / 2);
#define CK_K(LG) k_blk_from_i64<LG>
    CK_BLK13(CK_K, dim3(batch * limbs), m, out, limbs, tab_of(ctx));
#undef CK_K
    prof_end(ctx, K_NTT_FWD_ROW);
    HIP_TRY(hipGetLastError());
    return CKKS_OK;
}

ckks_status blk_encrypt(ckks_ctx *ctx, uint64_t *c0, uint64_t *c1, const uint64_t *a, const int8_t *s,
                        const int32_t *e, const uint64_t *m, uint32_t limbs)
{
    const double res = (double)limbs * ctx->n;
    prof_begin(ctx, K_NTT_FWD_ROW, 32.0 * res + 5.0 * ctx->n, res * kOpsButterflyF64 * ctx->log_n);
#define CK_K(LG) k_blk_encrypt<LG>
    CK_BLK13(CK_K, dim3(limbs), c0, c1, a, s, e, m, tab_of(ctx));
#undef CK_K
    prof_end(ctx, K_NTT_FWD_ROW);
    HIP_TRY(hipGetLastError());
    return CKKS_OK;
}

ckks_status blk_decrypt(ckks_ctx *ctx, uint64_t *pt, const uint64_t *c0, const uint64_t *c1, const int8_t *s,
                        uint32_t limbs)
{
    const double res = (double)limbs * ctx->n;
    prof_begin(ctx, K_NTT_FWD_ROW, 24.0 * res + ctx->n, res * kOpsButterflyF64 * ctx->log_n / 2);
#define CK_K(LG) k_blk_decrypt<LG>
    CK_BLK13(CK_K, dim3(limbs), pt, c0, c1, s, tab_of(ctx));
#undef CK_K
    prof_end(ctx, K_NTT_FWD_ROW);
    HIP_TRY(hipGetLastError());
    return CKKS_OK;
}

ckks_status blk_rescale(ckks_ctx *ctx, const uint64_t *c, uint32_t polys, uint32_t l, uint64_t *out, uint64_t *work)
{
    const Tab tb = tab_of(ctx);
    double *top = (double *)work;
    const ulonglong2 *qlinv = ctx->d_qlinv + (size_t)l * ctx->n_q;
    const double res = (double)polys * ctx->n, bf = kOpsButterflyF64 * ctx->log_n / 2;
    prof_begin(ctx, K_NTT_INV_ROW, 16.0 * res, res * bf);
#define CK_K(LG) k_blk_rescale_top<LG>
    CK_BLK(CK_K, dim3(polys), top, c, l, tb);
#undef CK_K
    prof_end(ctx, K_NTT_INV_ROW);
    HIP_TRY(hipGetLastError());
    prof_begin(ctx, K_NTT_FWD_ROW, 8.0 * res * (1 + 2.0 * l), res * l * bf);
#define CK_E(LG) k_blk_rescale<LG, (LG <= 13)>
#define CK_L(LG) k_blk_rescale<LG, false>
    CK_BLK_E((size_t)polys * l, dim3(polys * l), out, c, top, l, qlinv, tb);
#undef CK_E
#undef CK_L
    prof_end(ctx, K_NTT_FWD_ROW);
    HIP_TRY(hipGetLastError());
    return CKKS_OK;
}

ckks_status blk_modup(ckks_ctx *ctx, const uint64_t *c1, size_t stride, const uint64_t *b, uint32_t count,
                      uint32_t level, uint64_t *digits, uint64_t *stage)
{
    Digits dg{};
    dg.nd = n_digits(ctx, level);
    dg.alpha = ctx->alpha;
    dg.L = level + 1;
    dg.K = ctx->n_p;
    dg.n_q = ctx->n_q;
    for (uint32_t j = 0; j < dg.nd; j++) {
        const ConvDev *cd;
        CK_TRY(ctx_conv(ctx, (int)level, (int)j, &cd));
        dg.inv[j] = cd->d_qhat_inv_f;
        dg.mod[j] = cd->d_qhat_mod_f;
    }
    const uint32_t ext = dg.L + dg.K;
    const size_t N = ctx->n;
    const Tab tb = tab_of(ctx);
    double *y = (double *)stage;
    // a launch takes at most 65535 entries (blockIdx.y and z)
    for (uint32_t r0 = 0; r0 < count; r0 += 65535u) {
        const uint32_t cnt = std::min(count - r0, 65535u);
        const Source src{c1 + r0 * stride, stride, b};
        uint64_t *d = digits + (size_t)r0 * dg.nd * ext * N;
        double *yr = y + (size_t)r0 * dg.L * N;
        prof_begin(ctx, K_NTT_INV_ROW, 16.0 * cnt * dg.L * N);
#define CK_K(LG) k_blk_digits<LG, true>
        if (b) CK_BLK13(CK_K, dim3(dg.L, cnt), yr, src, dg, tb);
#undef CK_K
#define CK_K(LG) k_blk_digits<LG, false>
        if (!b) CK_BLK13(CK_K, dim3(dg.L, cnt), yr, src, dg, tb);
#undef CK_K
        prof_end(ctx, K_NTT_INV_ROW);
        HIP_TRY(hipGetLastError());
        prof_begin(ctx, K_CONV, 8.0 * cnt * N * (2.0 * dg.L + (double)dg.nd * ext));
        const size_t blocks = (size_t)ext * dg.nd * cnt;
#define CK_E(LG) k_blk_modup<LG, true, true>
#define CK_L(LG) k_blk_modup<LG, true, false>
        if (b) CK_BLK13_E(blocks, dim3(ext, dg.nd, cnt), d, yr, src, dg, tb);
#undef CK_E
#undef CK_L
#define CK_E(LG) k_blk_modup<LG, false, true>
#define CK_L(LG) k_blk_modup<LG, false, false>
        if (!b) CK_BLK13_E(blocks, dim3(ext, dg.nd, cnt), d, yr, src, dg, tb);
#undef CK_E
#undef CK_L
        prof_end(ctx, K_CONV);
        HIP_TRY(hipGetLastError());
    }
    return CKKS_OK;
}

ckks_status blk_rotate_batch(ckks_ctx *ctx, uint32_t level, const RotArgs &ra, uint64_t *work, const uint64_t *ta,
                             const uint64_t *tb2)
{
    const uint32_t L = level + 1, K = ctx->n_p, count = ra.count;
    const Tab tb = tab_of(ctx);
    const ConvDev *cd;
    CK_TRY(ctx_conv(ctx, (int)level, -1, &cd));
    CK_TRY(blk_key_product(ctx, level, ra, work));
    CK_TRY(launch_moddown_p(ctx, work, 2 * count, L, K, cd));
    prof_begin(ctx, K_MODDOWN, 8.0 * count * ctx->n * (2.0 * K + 7.0 * L));
    const dim3 grid(L, 2, count);
    const size_t blocks = (size_t)L * 2 * count;
#define CK_E(LG) k_blk_finish<LG, ADD_TENSOR, true>
#define CK_L(LG) k_blk_finish<LG, ADD_TENSOR, false>
    if (ta) CK_BLK13_E(blocks, grid, ra, work, L, K, cd->d_qhat_mod_f, ctx->d_pinv, ta, tb2, tb);
#undef CK_E
#undef CK_L
#define CK_E(LG) k_blk_finish<LG, ADD_ROWS, true>
#define CK_L(LG) k_blk_finish<LG, ADD_ROWS, false>
    if (!ta) CK_BLK13_E(blocks, grid, ra, work, L, K, cd->d_qhat_mod_f, ctx->d_pinv, ta, tb2, tb);
#undef CK_E
#undef CK_L
    prof_end(ctx, K_MODDOWN);
    HIP_TRY(hipGetLastError());
    return CKKS_OK;
}

ckks_status blk_moddown(ckks_ctx *ctx, uint64_t *u, uint32_t polys, uint32_t level, const uint64_t *add0,
                        uint32_t add0_g, const uint64_t *add1, uint64_t *out)
{
    const uint32_t L = level + 1, K = ctx->n_p;
    const Tab tb = tab_of(ctx);
    const ConvDev *cd;
    CK_TRY(ctx_conv(ctx, (int)level, -1, &cd));
    CK_REQUIRE(polys <= 65535u, CKKS_EINVAL, "moddown of %u polynomials in one call", polys);
    CK_TRY(launch_moddown_p(ctx, u, polys, L, K, cd));
    prof_begin(ctx, K_MODDOWN, 8.0 * polys * ctx->n * (K + 3.0 * L));
#define CK_E(LG) k_blk_moddown<LG, (LG <= 13)>
#define CK_L(LG) k_blk_moddown<LG, false>
    CK_BLK_E((size_t)L * polys, dim3(L, polys), out, u, add0, add0_g, add1, L, K, cd->d_qhat_mod_f, ctx->d_pinv, tb);
#undef CK_E
#undef CK_L
    prof_end(ctx, K_MODDOWN);
    HIP_TRY(hipGetLastError());
    return CKKS_OK;
}
