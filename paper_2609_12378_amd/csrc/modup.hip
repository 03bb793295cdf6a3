// ModUp and the conversion half of ModDown for rings of N >= 2^12 with fp64 arithmetic, two passes per transform
// (N1 x 256 points).
//
// A conversion Conv(x)_t = sum_i y_i [Qhat_i]_t starts from the centred digits y_i = [x_i Qhat_i^-1]: the inverse
// transform writes them itself, the constant folded into its last stage's factor N^-1.  A ModUp of any number of
// ciphertexts is four launches for all digits together at N = 2^16, five below:
//   1. row pass of the inverse transform of every limb, from the polynomial into the limb's row of its digit;
//   2. column pass, leaving the digits y there;
//   3. conversion of every digit, fused with the forward column pass where columns have 256 points;
//   4. forward row pass, which in the digits' own rows (no longer needed for y) puts the polynomial itself.
// One launch per digit and step and copies of the limbs in and out were 6 nd + 2 launches: an evaluation step with two
// key switches at N = 2^16 (13 limbs, two digits) took 378 us with those and 316 us so, 32 rotations sharing a ModUp
// (24 limbs, three digits) 1640 and 1536 us.
#include <algorithm>

#include "ckks_internal.h"
#include "ntt_core.h"
#include "ops.h"

namespace {

using A = nttc::Ar<true>;
using nttc::kE;
using nttc::kE8;

// The rows of `count` entries: entry r has nd blocks of `ext` rows, block j converts its own rows lo .. hi - 1
// (lo = j alpha, hi = min(lo + alpha, L)) to its other rows.  A ModUp: blocks are digits, rows 0 .. L - 1 are modulo
// q_row and L .. ext - 1 modulo the special primes.  A ModDown (down): one block of K = alpha = L = ext source rows
// modulo the special primes, converted to L_out rows elsewhere.
struct Blocks {
    uint32_t nd, alpha, L, ext, n_q;
    uint32_t log_n;
    bool down;
    uint32_t out_rows;                                   // rows of a block's output: ext, or L_out when down
    const double *inv[kMaxPrimes], *mod[kMaxPrimes];     // per block: Qhat_i^-1, and [Qhat_i]_t centred ([ns][nt])
    __device__ uint32_t lo(uint32_t j) const { return j * alpha; }
    __device__ uint32_t hi(uint32_t j) const { return min((j + 1) * alpha, L); }
    __device__ uint32_t src_prime(uint32_t l) const { return down ? n_q + l : l; }
    // target tt of block j: its row of the output, and that row's prime
    __device__ uint32_t out_row(uint32_t j, uint32_t tt) const { return down || tt < lo(j) ? tt : tt + hi(j) - lo(j); }
    __device__ uint32_t out_prime(uint32_t row) const { return down || row < L ? row : n_q + (row - L); }
    __device__ uint32_t targets(uint32_t j) const { return down ? out_rows : ext - (hi(j) - lo(j)); }
    // word offset of limb l's row in entry r
    __device__ size_t at(uint32_t r, uint32_t l) const { return ((size_t)(r * nd + l / alpha) * ext + l) << log_n; }
};

// 1. rows of 256 points, 8 per block of 128 threads: inverse row pass of limb l of c1 + r stride to its row
__global__ __launch_bounds__(128) void k_up_row(uint64_t *dst, const uint64_t *__restrict__ c1, size_t stride, Blocks bl,
                                                const ModQ *__restrict__ mods, const double *__restrict__ itwf)
{
    __shared__ double lds[8 * 273];
    const uint32_t n1 = 1u << (bl.log_n - 8), per = n1 / 8;
    const uint32_t row = blockIdx.x / per, r = row / bl.L, l = row % bl.L;
    const uint32_t sub = threadIdx.x >> 4, t = threadIdx.x & 15u, h = (blockIdx.x % per) * 8 + sub;
    const A ar(mods[l]);
    const double *tw = itwf + ((size_t)l << bl.log_n);
    const uint64_t *in = c1 + r * stride + ((size_t)l << bl.log_n) + (size_t)h * 256;
    uint64_t *out = dst + bl.at(r, l) + (size_t)h * 256;
    double x[kE];
#pragma unroll
    for (int k = 0; k < kE; k++) x[k] = A::from_u64(in[t + 16 * k]);
    nttc::transpose<8, true>(x, lds, sub, t);
    nttc::inv_low<8, true>(x, tw, n1 + h, t, ar);
    nttc::transpose<8, false>(x, lds, sub, t);
    nttc::inv_top<true>(x, tw, n1 + h, ar);
#pragma unroll
    for (int k = 0; k < kE; k++) out[t + 16 * k] = A::to_raw(x[k]);
}

// 2. inverse column pass of those rows, in place: the centred digits [x Qhat_l^-1] as doubles
template <int LOGS>
__global__ __launch_bounds__(256) void k_up_col(uint64_t *data, Blocks bl, const ModQ *__restrict__ mods,
                                                const double *__restrict__ itwf)
{
    constexpr uint32_t TS = (1u << LOGS) / 16, kCols = 4096u >> LOGS, kBpr = 256 / kCols;
    __shared__ double lds[LOGS > 4 ? kCols * ((1u << LOGS) + (1u << LOGS) / 16 + 1) : 1];
    const uint32_t row = blockIdx.x / kBpr, r = row / bl.L, l = row % bl.L, prime = bl.src_prime(l), j = l / bl.alpha;
    const A ar(mods[prime]);
    A sc = ar;  // N^-1 Qhat_l^-1
    sc.ninv = ar.scaled_twiddle(bl.inv[j][l - j * bl.alpha]);
    const double *tw = itwf + ((size_t)prime << bl.log_n);
    const uint32_t col = threadIdx.x % kCols, t = threadIdx.x / kCols;
    uint64_t *base = data + bl.at(r, l) + (blockIdx.x % kBpr) * kCols + col;
    double x[kE];
#pragma unroll
    for (int k = 0; k < kE; k++) x[k] = A::from_raw(base[(size_t)(LOGS > 4 ? 16 * t + k : k) * 256]);
    if (LOGS > 4) {
        nttc::inv_low<LOGS, true>(x, tw, 1, t, ar);
        nttc::transpose<LOGS, false>(x, lds, col, t);
    }
    nttc::inv_top<true, true>(x, tw, 1, sc);
#pragma unroll
    for (int k = 0; k < kE; k++) base[(size_t)(t + TS * k) * 256] = A::to_raw(ar.red(x[k]));
}

// 3. conversion alone (N1 < 256, or more than 8 sources): thread = one coefficient, blockIdx.y a group of t_per targets,
// blockIdx.z (entry, block); canonical residues out.  All loads issue before the first is used: short blocks repeat
// their last source.
template <int NS>
__global__ __launch_bounds__(256) void k_up_conv(uint64_t *out, const uint64_t *in, Blocks bl, uint32_t t_per,
                                                 const ModQ *__restrict__ mods)
{
    __shared__ double s_mod[NS * kMaxPrimes];
    __shared__ double2 s_tq[kMaxPrimes];
    const uint32_t j = blockIdx.z % bl.nd, r = blockIdx.z / bl.nd, lo = bl.lo(j);
    const int ns = (int)(bl.hi(j) - lo), nt = (int)bl.targets(j);
    const int t0 = (int)(blockIdx.y * t_per), t1 = min(nt, t0 + (int)t_per);
    if (t0 >= nt) return;
    for (int k = threadIdx.x; k < ns * (t1 - t0); k += 256)
        s_mod[k] = bl.mod[j][(k / (t1 - t0)) * nt + t0 + k % (t1 - t0)];
    for (int k = threadIdx.x; k < t1 - t0; k += 256) {
        const ModQ &m = mods[bl.out_prime(bl.out_row(j, t0 + k))];
        s_tq[k] = make_double2(m.qd, m.qinvd);
    }
    const uint32_t col = blockIdx.x * 256 + threadIdx.x;
    const uint64_t *src = in + bl.at(r, lo) + col;
    double y[NS];
#pragma unroll
    for (int i = 0; i < NS; i++) y[i] = A::from_raw(src[(size_t)min(i, ns - 1) << bl.log_n]);
    __syncthreads();
    uint64_t *dst = out + ((size_t)(r * bl.nd + j) * bl.out_rows << bl.log_n) + col;
    for (int t = t0; t < t1; t++) {
        A ar;
        ar.q = s_tq[t - t0].x;
        ar.qinv = s_tq[t - t0].y;
        nttc::GridSum acc;
#pragma unroll
        for (int i = 0; i < NS; i++) {
            if (i < ns) {
                acc.add(y[i], s_mod[i * (t1 - t0) + (t - t0)]);
                if ((i & 7) == 7 && i + 1 < ns) acc.fold(ar);
            }
        }
        dst[(size_t)bl.out_row(j, t) << bl.log_n] = ar.to_canon(acc.value(ar));
    }
}

// 3. the conversion (at most 8 sources) fused with the first forward column pass, N = 2^16: block (entry, 16 adjacent
// columns; group of t_per targets; block j of the entry), 512 threads, 8 points of one 256-point column per thread.
// The source digits of the block's 4096 coefficients stay in registers; for each target in turn the block forms the
// converted residues (one quotient per eight-term sum, nttc::GridSum, reduced to |x| <= t/2), runs that limb's column
// sub-transforms on them (nttc::fwd8_256_loop with the column pass's lazy-reduction mask) and writes the rows as raw
// doubles, the inter-pass form the row passes read.  The converted rows thus cross HBM once instead of three times.
// Target t + 1's twiddles (Psi[1..255]) are staged into the idle half of a double-buffered table while target t is
// transformed.  EXACT: every block has 8 sources.  32 rotations at 24 limbs: 600 us with a reduced product per term and
// the digits formed here, 550 us with the one quotient, 505 us from ready digits; with 212 registers it runs two
// waves a SIMD.  Blocks of 8 columns (256 threads, two independent blocks a CU) measured the same within 1% on every
// call, so the two barriers per target are not what bounds it: the fp64 pipes at their sustained clock are.
template <bool EXACT>
__global__ __launch_bounds__(512) void k_conv_col8(uint64_t *out, const uint64_t *in, Blocks bl, uint32_t t_per,
                                                   const ModQ *__restrict__ mods, const double *__restrict__ twf)
{
    __shared__ double s_mod[8 * kMaxPrimes];
    __shared__ double tws[2][256];
    __shared__ double tr[16][nttc::kTr8], trb[16][nttc::kTr8];
    constexpr uint32_t log_n = 16, n2 = 256;
    const uint32_t r = blockIdx.x >> 4, blk = blockIdx.x & 15u, j = blockIdx.z, lo = bl.lo(j);
    const int ns = EXACT ? 8 : (int)(bl.hi(j) - lo), nt = (int)bl.targets(j);
    const int t0 = (int)(blockIdx.y * t_per), t1 = min(nt, t0 + (int)t_per);
    if (t0 >= nt) return;
    for (int k = threadIdx.x; k < ns * nt; k += 512) s_mod[k] = bl.mod[j][k];
    if (threadIdx.x < 255)
        tws[t0 & 1][threadIdx.x + 1] = twf[((size_t)bl.out_prime(bl.out_row(j, t0)) << log_n) + threadIdx.x + 1];
    const uint32_t col = threadIdx.x & 15, t = threadIdx.x >> 4;
    const uint32_t coff = blk * 16 + col;
    const uint64_t *src = in + bl.at(r, lo) + coff;
    double y[8][kE8];
#pragma unroll
    for (int i = 0; i < 8; i++)
#pragma unroll
        for (int k = 0; k < kE8; k++)
            if (EXACT || i < ns) y[i][k] = A::from_raw(src[((size_t)i << log_n) + (size_t)nttc::u8<0>(t, k) * n2]);
    uint64_t *dst0 = out + ((size_t)(r * bl.nd + j) * bl.out_rows << log_n) + coff;
    __syncthreads();
    for (int tt = t0; tt < t1; tt++) {
        const uint32_t row = bl.out_row(j, tt);
        const A ar(mods[bl.out_prime(row)]);
        nttc::StageNext next{tws[(tt + 1) & 1], 0.0, tt + 1 < t1 && threadIdx.x < 255};
        if (next.on) next.v = twf[((size_t)bl.out_prime(bl.out_row(j, tt + 1)) << log_n) + threadIdx.x + 1];
        double x[kE8];
#pragma unroll
        for (int k = 0; k < kE8; k++) {
            nttc::GridSum acc;
#pragma unroll
            for (int i = 0; i < 8; i++)
                if (EXACT || i < ns) acc.add(y[i][k], s_mod[i * nt + tt]);
            x[k] = ar.red(acc.value(ar));
        }
        nttc::fwd8_256_loop<nttc::kColMask8>(x, tws[tt & 1], tr[col], trb[col], t, ar, next);
        uint64_t *dst = dst0 + ((size_t)row << log_n);
#pragma unroll
        for (int k = 0; k < kE8; k++) nttc::st_stream(dst + (size_t)nttc::u8<2>(t, k) * n2, A::to_raw(x[k]));
    }
}

// masks of the forward stages that reduce (ntt.hip: column output below 2 q, or below 4.3 q from k_conv_col8)
constexpr unsigned up_col_mask(int logs)
{
    return logs == 4 ? 0x0c : logs == 5 ? 0x1c : logs == 6 ? 0x34 : logs == 7 ? 0x74 : 0xd4;
}

// 3b. forward column pass of the converted rows, own rows left alone
template <int LOGS>
__global__ __launch_bounds__(256) void k_up_fcol(uint64_t *data, Blocks bl, const ModQ *__restrict__ mods,
                                                 const double *__restrict__ twf)
{
    constexpr uint32_t TS = (1u << LOGS) / 16, kCols = 4096u >> LOGS, kBpr = 256 / kCols;
    __shared__ double lds[LOGS > 4 ? kCols * ((1u << LOGS) + (1u << LOGS) / 16 + 1) : 1];
    const uint32_t rr = blockIdx.x / kBpr, row = rr % bl.ext, b = rr / bl.ext, j = b % bl.nd;
    if (row >= bl.lo(j) && row < bl.hi(j)) return;
    const uint32_t prime = bl.out_prime(row);
    const A ar(mods[prime]);
    const double *tw = twf + ((size_t)prime << bl.log_n);
    const uint32_t col = threadIdx.x % kCols, t = threadIdx.x / kCols;
    uint64_t *base = data + ((size_t)rr << bl.log_n) + (blockIdx.x % kBpr) * kCols + col;
    double x[kE];
#pragma unroll
    for (int k = 0; k < kE; k++) x[k] = A::from_u64(base[(size_t)(t + TS * k) * 256]);
    constexpr unsigned kMask = up_col_mask(LOGS);
    nttc::fwd_top<true, kMask>(x, tw, 1, ar);
    if (LOGS > 4) {
        nttc::transpose<LOGS, true>(x, lds, col, t);
        nttc::fwd_low<LOGS, true, kMask>(x, tw, 1, t, ar);
    }
#pragma unroll
    for (int k = 0; k < kE; k++) base[(size_t)(LOGS > 4 ? 16 * t + k : k) * 256] = A::to_raw(x[k]);
}

// 4. forward row pass, canonical out; a digit's own rows take the polynomial's.  Input below 4.3 q: stages 0, 2, 4, 6
// reducing keep every value below 7 q.
constexpr unsigned kUpRowMask = 0x55;
__global__ __launch_bounds__(128) void k_up_frow(uint64_t *data, const uint64_t *__restrict__ c1, size_t stride,
                                                 Blocks bl, const ModQ *__restrict__ mods,
                                                 const double *__restrict__ twf)
{
    __shared__ double lds[8 * 273];
    const uint32_t n1 = 1u << (bl.log_n - 8), per = n1 / 8;
    const uint32_t rr = blockIdx.x / per, row = rr % bl.ext, b = rr / bl.ext, j = b % bl.nd, r = b / bl.nd;
    const uint32_t sub = threadIdx.x >> 4, t = threadIdx.x & 15u, h = (blockIdx.x % per) * 8 + sub;
    uint64_t *base = data + ((size_t)rr << bl.log_n) + (size_t)h * 256;
    if (row >= bl.lo(j) && row < bl.hi(j)) {
        const uint64_t *in = c1 + r * stride + ((size_t)row << bl.log_n) + (size_t)h * 256;
        uint64_t v[kE];
#pragma unroll
        for (int k = 0; k < kE; k++) v[k] = in[t + 16 * k];
#pragma unroll
        for (int k = 0; k < kE; k++) base[t + 16 * k] = v[k];
        return;
    }
    const uint32_t prime = bl.out_prime(row);
    const A ar(mods[prime]);
    const double *tw = twf + ((size_t)prime << bl.log_n);
    double x[kE];
#pragma unroll
    for (int k = 0; k < kE; k++) x[k] = A::from_raw(base[t + 16 * k]);
    nttc::fwd_top<true, kUpRowMask>(x, tw, n1 + h, ar);
    nttc::transpose<8, true>(x, lds, sub, t);
    nttc::fwd_low<8, true, kUpRowMask>(x, tw, n1 + h, t, ar);
    nttc::transpose<8, false>(x, lds, sub, t);
#pragma unroll
    for (int k = 0; k < kE; k++) base[t + 16 * k] = ar.to_canon(x[k]);
}

ckks_status launch_col_digits(ckks_ctx *ctx, uint64_t *data, uint32_t count, const Blocks &bl)
{
    const uint32_t rows = count * bl.L;
    prof_begin(ctx, K_NTT_INV_COL, 16.0 * rows * ctx->n, (double)rows * ctx->n * kOpsButterflyF64 * (ctx->log_n - 8) / 2);
#define CK_COL(S)                                                                                                  \
    hipLaunchKernelGGL(k_up_col<S>, dim3(rows * (256 / (4096u >> S))), dim3(256), 0, ctx->stream, data, bl, ctx->d_mod, \
                       ctx->d_itwf)
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

// columns of 256 points and few enough sources for the registers of the fused conversion
bool conv_fused(const ckks_ctx *ctx, uint32_t max_src) { return ctx->log_n == 16 && max_src <= 8; }

// the conversion of every block of `count` entries; max_src, max_tgt over the blocks
ckks_status launch_blocks_conv(ckks_ctx *ctx, uint64_t *out, const uint64_t *in, uint32_t count, const Blocks &bl,
                               uint32_t max_src, uint32_t max_tgt, bool exact8)
{
    const double res = (double)count * bl.nd * ctx->n;
    prof_begin(ctx, K_CONV, 8.0 * res * (max_src + max_tgt),
               res * max_tgt * (max_src * 4.0 + 7.0 + (conv_fused(ctx, max_src) ? kOpsButterflyF64 * 4 : 0.0)));
    if (conv_fused(ctx, max_src)) {
        // fewer than 256 blocks (one a CU): the targets split over blockIdx.y until the grid has that many
        const uint32_t blocks = count * 16 * bl.nd, groups = std::min(max_tgt, std::max(1u, 256u / blocks));
        const uint32_t t_per = (max_tgt + groups - 1) / groups;
        const dim3 grid(count * 16, (max_tgt + t_per - 1) / t_per, bl.nd);
        if (exact8)
            hipLaunchKernelGGL(k_conv_col8<true>, grid, dim3(512), 0, ctx->stream, out, in, bl, t_per, ctx->d_mod,
                               ctx->d_twf);
        else
            hipLaunchKernelGGL(k_conv_col8<false>, grid, dim3(512), 0, ctx->stream, out, in, bl, t_per, ctx->d_mod,
                               ctx->d_twf);
    } else {
        // groups of targets until the grid has 2048 blocks of four waves (two waves a SIMD)
        for (uint32_t r0 = 0; r0 < count; r0 += 65535u / bl.nd) {
            const uint32_t cnt = std::min(count - r0, 65535u / bl.nd);
            const uint32_t blocks = cnt * bl.nd * (ctx->n / 256);
            const uint32_t groups = std::min(max_tgt, std::max(1u, 2048u / blocks));
            const uint32_t t_per = (max_tgt + groups - 1) / groups;
            const dim3 grid(ctx->n / 256, (max_tgt + t_per - 1) / t_per, cnt * bl.nd);
            const size_t e = (size_t)r0 * bl.nd * ctx->n;
            if (max_src <= 8)
                hipLaunchKernelGGL(k_up_conv<8>, grid, dim3(256), 0, ctx->stream, out + e * bl.out_rows, in + e * bl.ext,
                                   bl, t_per, ctx->d_mod);
            else
                hipLaunchKernelGGL(k_up_conv<16>, grid, dim3(256), 0, ctx->stream, out + e * bl.out_rows,
                                   in + e * bl.ext, bl, t_per, ctx->d_mod);
        }
    }
    prof_end(ctx, K_CONV);
    HIP_TRY(hipGetLastError());
    return CKKS_OK;
}

}  // namespace

bool up_conv_ok(const ckks_ctx *ctx, const ConvDev *cd)
{
    return ctx->log_n >= 12 && cd->f64 && cd->ns >= 1 && cd->ns <= 16;
}

bool f64_level_ok(const ckks_ctx *ctx, uint32_t level)
{
    if (!ctx->n_p) return false;
    for (uint32_t i = 0; i < ctx->n_primes(); i++)
        if ((i <= level || i >= ctx->n_q) && !ctx->f64_ok[i]) return false;
    for (int j = -1; j < (int)n_digits(ctx, level); j++) {
        const auto it = ctx->conv.find({(int)level, j});
        if (it == ctx->conv.end() || !up_conv_ok(ctx, &it->second)) return false;
    }
    return true;
}

ckks_status up_modup(ckks_ctx *ctx, const uint64_t *c1, size_t stride, uint32_t count, uint32_t level, uint64_t *digits)
{
    Blocks bl{};
    bl.nd = n_digits(ctx, level);
    bl.alpha = ctx->alpha;
    bl.L = level + 1;
    bl.ext = bl.out_rows = bl.L + ctx->n_p;
    bl.n_q = ctx->n_q;
    bl.log_n = ctx->log_n;
    uint32_t max_src = 0, max_tgt = 0;
    bool exact8 = true;
    for (uint32_t j = 0; j < bl.nd; j++) {
        const ConvDev *cd;
        CK_TRY(ctx_conv(ctx, (int)level, (int)j, &cd));
        bl.inv[j] = cd->d_qhat_inv_f;
        bl.mod[j] = cd->d_qhat_mod_f;
        max_src = std::max(max_src, (uint32_t)cd->ns);
        max_tgt = std::max(max_tgt, (uint32_t)cd->nt);
        exact8 = exact8 && cd->ns == 8;
    }
    const uint32_t per = 1u << (ctx->log_n - 11);  // blocks of eight 256-point rows
    const double res = (double)count * bl.L * ctx->n;
    prof_begin(ctx, K_NTT_INV_ROW, 16.0 * res, res * kOpsButterflyF64 * 4);
    hipLaunchKernelGGL(k_up_row, dim3(count * bl.L * per), dim3(128), 0, ctx->stream, digits, c1, stride, bl, ctx->d_mod,
                       ctx->d_itwf);
    prof_end(ctx, K_NTT_INV_ROW);
    HIP_TRY(hipGetLastError());
    CK_TRY(launch_col_digits(ctx, digits, count, bl));
    CK_TRY(launch_blocks_conv(ctx, digits, digits, count, bl, max_src, max_tgt, exact8));
    const uint32_t rows = count * bl.nd * bl.ext;
    if (!conv_fused(ctx, max_src)) {
        prof_begin(ctx, K_NTT_FWD_COL, 16.0 * rows * ctx->n);
#define CK_COL(S)                                                                                                  \
    hipLaunchKernelGGL(k_up_fcol<S>, dim3(rows * (256 / (4096u >> S))), dim3(256), 0, ctx->stream, digits, bl,       \
                       ctx->d_mod, ctx->d_twf)
        switch (ctx->log_n) {
        case 12: CK_COL(4); break;
        case 13: CK_COL(5); break;
        case 14: CK_COL(6); break;
        case 15: CK_COL(7); break;
        default: CK_COL(8); break;
        }
#undef CK_COL
        prof_end(ctx, K_NTT_FWD_COL);
        HIP_TRY(hipGetLastError());
    }
    prof_begin(ctx, K_NTT_FWD_ROW, 16.0 * rows * ctx->n, (double)rows * ctx->n * kOpsButterflyF64 * 4);
    hipLaunchKernelGGL(k_up_frow, dim3(rows * per), dim3(128), 0, ctx->stream, digits, c1, stride, bl, ctx->d_mod,
                       ctx->d_twf);
    prof_end(ctx, K_NTT_FWD_ROW);
    HIP_TRY(hipGetLastError());
    return CKKS_OK;
}

ckks_status up_moddown(ckks_ctx *ctx, uint64_t *up, uint32_t polys, uint32_t level, uint64_t *cw)
{
    const ConvDev *cd;
    CK_TRY(ctx_conv(ctx, (int)level, -1, &cd));
    Blocks bl{};
    bl.nd = 1;
    bl.alpha = bl.L = bl.ext = ctx->n_p;
    bl.n_q = ctx->n_q;
    bl.log_n = ctx->log_n;
    bl.down = true;
    bl.out_rows = level + 1;
    bl.inv[0] = cd->d_qhat_inv_f;
    bl.mod[0] = cd->d_qhat_mod_f;
    CK_TRY(launch_col_digits(ctx, up, polys, bl));
    CK_TRY(launch_blocks_conv(ctx, cw, up, polys, bl, ctx->n_p, level + 1, ctx->n_p == 8));
    if (!conv_fused(ctx, ctx->n_p))
        CK_TRY(launch_ntt_fwd_first_pass(ctx, cw, polys, level + 1, limb_range(0, level + 1)));
    return CKKS_OK;
}
