// The whole negacyclic transform of one row of N = 2^12 .. 2^14 residues inside one block (fp64 arithmetic).
//
// The factorisation is that of the two-pass transform (ntt.hip): index x = 256 h + c, columns of N1 = N / 256 points
// (stages that mix h, twiddle base 1), then rows of 256 points (base N1 + h), 16 residues a thread, N / 16 threads.
// Between the two the row crosses LDS instead of HBM (34, 72 or 141 KB of the CU's 160), so a kernel that forms the
// row in registers, transforms it and consumes the result in registers does in one launch what the two passes do in
// two with an element-wise kernel on either side.  A row's 256 points belong to 16 lanes of one wave, so the row
// part needs no block barrier: the forward transform has one (N = 2^12) or three.
// Layouts (thread t, register k):
//   column: x[k] is point (r + TS1 k) * 256 + c with c = t mod 256, r = t / 256, TS1 = N1 / 16;
//   row:    x[k] is point 256 h + (t mod 16) + 16 k with h = t / 16.
// In both, consecutive lanes hold consecutive points (runs of 16 in the row layout), so global accesses of either
// are whole 128-byte segments.
//
// With a few rows a launch lasts as long as its chain of memory round trips (L2 holds nothing of the previous kernel
// on gfx950's eight dies, so each is about a microsecond): a transform that loads a stage's twiddles when it comes to
// the stage takes nine.  Twiddles therefore are loaded together, up front, into registers: the columns' are the same
// for a whole wave (scalar loads, ColTw), a thread's 30 for its row are 60 VGPRs (RowTw).
#pragma once
#include "ntt_core.h"

namespace blk {

using A = nttc::Ar<true>;
using nttc::kE;

constexpr int kMinLog = 12, kMaxLog = 14;
template <int LOGN>
struct Shape {
    static constexpr int S1 = LOGN - 8;
    static constexpr uint32_t N1 = 1u << S1, TS1 = N1 / 16, NT = 1u << (LOGN - 4);
    // padded words: the columns' transpose (N1 > 16) or the rows
    static constexpr uint32_t kCols = 256u * (N1 + N1 / 16 + 1), kRows = N1 * 272u;
    static constexpr uint32_t kLds = S1 > 4 && kCols > kRows ? kCols : kRows;
};

// masks of the forward stages that reduce: those of the two passes (column output below 2 q)
constexpr unsigned col_mask(int s1) { return s1 == 4 ? 0x0c : s1 == 5 ? 0x1c : 0x34; }
constexpr unsigned kRowMask = 0x54;

// LDS word of point u of row h: a word of padding every 16 and rows 16 mod 32 words apart, so that of the two rows
// that half a wave reads or writes (strides 1 and 17 between its 16 lanes) each takes the other's 32-word banks
__device__ __forceinline__ uint32_t ridx(uint32_t h, uint32_t u) { return h * 272u + u + (u >> 4); }

// the row transposes exchange data among the 16 lanes that hold one row: LDS accesses of a wave complete in order,
// so only the compiler has to keep the order
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
template <bool A_TOP>
__device__ __forceinline__ void row_transpose(double (&x)[kE], double *lds, uint32_t h, uint32_t r)
{
#pragma unroll
    for (int k = 0; k < kE; k++) lds[ridx(h, A_TOP ? r + 16 * k : 16 * r + k)] = x[k];
    wave_sync();
#pragma unroll
    for (int k = 0; k < kE; k++) x[k] = lds[ridx(h, A_TOP ? 16 * r + k : r + 16 * k)];
    wave_sync();
}

template <int LOGN>
__device__ __forceinline__ uint32_t col_pos(uint32_t t, int k)
{
    return ((t >> 8) + Shape<LOGN>::TS1 * (uint32_t)k) * 256u + (t & 255u);
}
__device__ __forceinline__ uint32_t row_pos(uint32_t t, int k) { return (t >> 4) * 256u + (t & 15u) + 16u * (uint32_t)k; }

// read-only tables that no kernel writes: loads the compiler may issue at any point, scalar where the index is
// uniform
template <typename T>
using Const = const __attribute__((address_space(4))) T *;
template <typename T>
__device__ __forceinline__ Const<T> as_const(const T *p)
{
    return (Const<T>)p;
}

// column twiddles Psi[1..15] and, for N1 > 16, those of the remaining stages of this wave's points 16 r ..
template <int LOGN>
struct ColTw {
    static constexpr int kLow = Shape<LOGN>::S1 == 4 ? 1 : Shape<LOGN>::S1 == 5 ? 8 : 12;
    double top[15], low[kLow];
    __device__ explicit ColTw(const double *tw)
    {
        const Const<double> c = as_const(tw);
#pragma unroll
        for (int i = 0; i < 15; i++) top[i] = c[1 + i];
        if constexpr (Shape<LOGN>::S1 > 4) {
            const uint32_t r = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
            int n = 0;
#pragma unroll
            for (int l = 0; l < Shape<LOGN>::S1 - 4; l++) {
                const int mp = 16 << l, gpt = 8 / ((int)Shape<LOGN>::N1 / (2 * mp));
#pragma unroll
                for (int g = 0; g < gpt; g++) low[n++] = c[mp + r * gpt + g];
            }
        }
    }
};
// this thread's row twiddles: Psi[B m + g] (m = 1, 2, 4, 8; g < m), then Psi[B m + g'] of its points' groups
// (m = 16 .. 128), B = N1 + h
template <int LOGN>
struct RowTw {
    double top[15], low[15];
    __device__ explicit RowTw(const double *tw)
    {
        const Const<double> c = as_const(tw);
        const uint32_t B = Shape<LOGN>::N1 + (threadIdx.x >> 4), r = threadIdx.x & 15u;
#pragma unroll
        for (int l = 0; l < 4; l++)
#pragma unroll
            for (int g = 0; g < 1 << l; g++) {
                top[(1 << l) - 1 + g] = c[(B << l) + g];
                low[(1 << l) - 1 + g] = c[(B << (4 + l)) + (r << l) + g];
            }
    }
};

// forward: the top four stages (x[k] is point r + TS k) and the stages after them (x[k] is point 16 r + k), for a
// sub-transform of 2^LOGS points
template <unsigned RMASK>
__device__ __forceinline__ void fwd_top(double (&x)[kE], const double (&w)[15], const A &ar)
{
#pragma unroll
    for (int l = 0; l < 4; l++) {
        const int tk = 8 >> l;
#pragma unroll
        for (int g = 0; g < 1 << l; g++)
#pragma unroll
            for (int j = 0; j < tk; j++)
                nttc::ct_stage<true, RMASK>(ar, l, x[g * 2 * tk + j], x[g * 2 * tk + j + tk], w[(1 << l) - 1 + g]);
    }
}
template <int LOGS, unsigned RMASK, int NW>
__device__ __forceinline__ void fwd_low(double (&x)[kE], const double (&w)[NW], const A &ar)
{
    int n = 0;
#pragma unroll
    for (int l = 0; l < LOGS - 4; l++) {
        const int t = (1 << LOGS) / (32 << l), gpt = 8 / t;
#pragma unroll
        for (int g = 0; g < gpt; g++, n++)
#pragma unroll
            for (int j = 0; j < t; j++)
                nttc::ct_stage<true, RMASK>(ar, 4 + l, x[g * 2 * t + j], x[g * 2 * t + j + t], w[n]);
    }
}
template <int LOGS, int NW>
__device__ __forceinline__ void inv_low(double (&x)[kE], const double (&w)[NW], const A &ar)
{
    int n = NW;
    if (LOGS == 4) n = 0;
#pragma unroll
    for (int l = LOGS - 5; l >= 0; l--) {
        const int t = (1 << LOGS) / (32 << l), gpt = 8 / t;
        n -= gpt;
#pragma unroll
        for (int g = 0; g < gpt; g++)
#pragma unroll
            for (int j = 0; j < t; j++) ar.gs(x[g * 2 * t + j], x[g * 2 * t + j + t], w[n + g]);
    }
}
// the last stage scaled (Ar<true>::gs_scaled with ar_scale's factor) if SCALED
template <bool SCALED>
__device__ __forceinline__ void inv_top(double (&x)[kE], const double (&w)[15], const A &ar, const A &ar_scale)
{
#pragma unroll
    for (int l = 3; l >= (SCALED ? 1 : 0); l--) {
        const int tk = 8 >> l;
#pragma unroll
        for (int g = 0; g < 1 << l; g++)
#pragma unroll
            for (int j = 0; j < tk; j++) ar.gs(x[g * 2 * tk + j], x[g * 2 * tk + j + tk], w[(1 << l) - 1 + g]);
    }
    if (SCALED) {
        const double wn = ar_scale.scaled_twiddle(w[0]);
#pragma unroll
        for (int j = 0; j < 8; j++) ar_scale.gs_scaled(x[j], x[j + 8], wn);
    }
}

// column layout in (|x| <= q), row layout out (|x| < 4.1 q).  Block barriers: every thread calls it; lds is free to be
// written by any thread on entry and only holds words of this thread's own row on exit.
template <int LOGN>
__device__ __forceinline__ void forward(double (&x)[kE], double *lds, const ColTw<LOGN> &cw, const RowTw<LOGN> &rw,
                                        const A &ar)
{
    using S = Shape<LOGN>;
    const uint32_t t = threadIdx.x, c = t & 255u, r = t >> 8;
    constexpr unsigned kCol = col_mask(S::S1);
    fwd_top<kCol>(x, cw.top, ar);
    if constexpr (S::S1 > 4) {
        nttc::transpose<S::S1, true>(x, lds, c, r);
        fwd_low<S::S1, kCol>(x, cw.low, ar);
    }
#pragma unroll
    for (int k = 0; k < kE; k++) lds[ridx(S::S1 > 4 ? 16 * r + k : k, c)] = x[k];
    __syncthreads();
    const uint32_t h = t >> 4, r2 = t & 15u;
    // from here on a thread touches only words of its own row, which 16 lanes of its wave share
#pragma unroll
    for (int k = 0; k < kE; k++) x[k] = lds[ridx(h, r2 + 16 * k)];
    wave_sync();
    fwd_top<kRowMask>(x, rw.top, ar);
    row_transpose<true>(x, lds, h, r2);
    fwd_low<8, kRowMask>(x, rw.low, ar);
    row_transpose<false>(x, lds, h, r2);
}

// row layout in (|x| < 2 q), column layout out: the inverse transform times ar_scale.ninv, |x| < 2 q (ar_scale is ar
// with the factor, N^-1 mod q times whatever the caller folds in, in its ninv)
template <int LOGN>
__device__ __forceinline__ void inverse(double (&x)[kE], double *lds, const ColTw<LOGN> &cw, const RowTw<LOGN> &rw,
                                        const A &ar, const A &ar_scale)
{
    using S = Shape<LOGN>;
    const uint32_t t = threadIdx.x, c = t & 255u, r = t >> 8;
    const uint32_t h = t >> 4, r2 = t & 15u;
    row_transpose<true>(x, lds, h, r2);
    inv_low<8>(x, rw.low, ar);
    row_transpose<false>(x, lds, h, r2);
    inv_top<false>(x, rw.top, ar, ar);
#pragma unroll
    for (int k = 0; k < kE; k++) lds[ridx(h, r2 + 16 * k)] = x[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kE; k++) x[k] = lds[ridx(S::S1 > 4 ? 16 * r + k : k, c)];
    if constexpr (S::S1 > 4) {
        inv_low<S::S1>(x, cw.low, ar);
        __syncthreads();
        nttc::transpose<S::S1, false>(x, lds, c, r);
    }
    inv_top<true>(x, cw.top, ar, ar_scale);
}

}  // namespace blk
