// The paper's preconditioner M = F^-1 D F (Section 3.2), applied to an l x c
// image zero-embedded in a P x P grid, with D = h(|omega|) of eq. (3.2) on the
// radial frequency.  Three kernels:
//
//  1. rows forward: two real rows are packed as one complex row (real and
//     imaginary parts), transformed, and split into the two half spectra
//     u = 0..P/2 (Hermitian symmetry) -> scratch S[l][P/2+1];
//  2. columns: NF half-spectrum columns per workgroup; forward FFT over the P
//     rows (rows >= l are the zero embedding), multiply by D(u, v), inverse FFT,
//     keep rows < l;
//  3. rows inverse: two rows rebuilt from their half spectra as one complex
//     row, inverse FFT; real part -> row r, imaginary part -> row r+1; crop to c
//     columns.
//
// The output is real because D is real and even in both frequencies.
// Arithmetic and scratch are float64 (input and output float32, in the solvers
// float64): with mu = 1e-5 the window spans five decades, and a float32
// transform's rounding swamps the low-frequency part of z.
//
// Transforms.  A thread keeps eight elements in registers and the passes are
// radix 8 (the last one 2, 4 or 8), self-sorting: natural order in and out, an
// exchange through LDS between passes.  Bound: latency (one 512^2 image has
// about one wave per SIMD; of the column kernel's 12.6 us about 6 are the two
// transforms' chains of LDS round trips, barriers and butterflies, 3 its loads
// and stores of single columns), so what counts is the number of steps in a row:
// P = 1024 takes 3 exchanges where radix-2 stages taken in pairs through LDS
// took 5 and a bit-reversed scatter, the next pass's twiddles are loaded before
// the exchange (as separate loads in each branch they cost a trip to L2 each),
// and the window and the inverse's first pass start from the registers the
// forward one ends in.  At 2048^2 the registers count too: up to 128, so that
// two workgroups of a CU overlap (188: 176 us, 126: 139).  z = M g, before and now:
// 64^2 18.1 -> 13.4 us, 243^2 23.0 -> 15.0, 512^2 35.4 -> 23.7, 1024^2 86.6 ->
// 49.7, 2048^2 295 -> 139; in 16 slices of 128^2 to 512^2 128 -> 71.
#include "sp_internal.h"
#include "sp_reduce.h"

#include <algorithm>

namespace sp {

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}

__device__ __forceinline__ double2 cadd(double2 a, double2 b) {
    return make_double2(a.x + b.x, a.y + b.y);
}
__device__ __forceinline__ double2 csub(double2 a, double2 b) {
    return make_double2(a.x - b.x, a.y - b.y);
}

// Transform elements per thread.
constexpr int FE = 8;

// This thread's elements of the workgroup's blockDim.x * FE / P transforms:
// register k holds position pos(k) of transform col(k).  P >= FE: P / FE threads
// per transform, positions t + k P / FE; with IL neighbouring threads hold
// neighbouring transforms (columns, which lie side by side in memory), else
// neighbouring positions.  SMALL (P < FE): FE / P transforms per thread.
template <bool IL, bool SMALL>
struct FftLane {
    int logP, t, c, lc;

    __device__ __forceinline__ explicit FftLane(int lp) : logP(lp) {
        const int tid = threadIdx.x;
        lc = 31 - __builtin_clz(blockDim.x * FE) - logP;   // log2 of the transforms
        if (SMALL) {
            t = tid;
            c = 0;
        } else if (IL) {
            c = tid & ((1 << lc) - 1);
            t = tid >> lc;
        } else {
            t = tid & ((1 << (logP - 3)) - 1);
            c = tid >> (logP - 3);
        }
    }
    __device__ __forceinline__ int pos(int k) const { return SMALL ? k >> (3 - logP) : t + (k << (logP - 3)); }
    __device__ __forceinline__ int col(int k) const {
        return SMALL ? (t << (3 - logP)) + (k & ((FE >> logP) - 1)) : c;
    }
    // Registers up to this one hold the lower half of the positions, where a
    // zero-embedded row or column lies.
    static constexpr int LOWER = SMALL ? FE : FE / 2;
    // LDS slot of position p of transform q.  The low bits are permuted by the
    // position's, so that the first exchange's writes, FE positions apart, do not
    // pile onto the same banks.
    __device__ __forceinline__ int slot(int p, int q) const {
        return IL ? ((p << lc) + q) ^ (((p >> 3) << lc) & 7) : ((q << logP) + p) ^ ((p >> 3) & 7);
    }
};

__device__ __forceinline__ double2 mul_mi(double2 a) { return make_double2(a.y, -a.x); }   // -i a

__device__ __forceinline__ void dft2(double2& a, double2& b) {
    const double2 t = a;
    a = cadd(t, b);
    b = csub(t, b);
}
// exp(-i) DFTs of 4 values in natural order.
__device__ __forceinline__ void dft4(double2& a, double2& b, double2& c, double2& d) {
    dft2(a, c);
    dft2(b, d);
    const double2 e = mul_mi(d);
    const double2 y1 = cadd(c, e), y3 = csub(c, e);
    dft2(a, b);   // y0, y2
    const double2 y2 = b;
    b = y1;
    c = y2;
    d = y3;
}
// ... and of 8.
__device__ __forceinline__ void dft8(double2 (&v)[FE]) {
    constexpr double R = 0.70710678118654752440;   // sqrt(1/2)
#pragma unroll
    for (int k = 0; k < 4; ++k) dft2(v[k], v[k + 4]);
    v[5] = make_double2((v[5].x + v[5].y) * R, (v[5].y - v[5].x) * R);
    v[6] = mul_mi(v[6]);
    v[7] = make_double2((v[7].y - v[7].x) * R, -(v[7].x + v[7].y) * R);
    dft4(v[0], v[1], v[2], v[3]);   // outputs 0, 2, 4, 6
    dft4(v[4], v[5], v[6], v[7]);   // outputs 1, 3, 5, 7
    const double2 y1 = v[4], y2 = v[1], y3 = v[5], y4 = v[2], y5 = v[6], y6 = v[3];
    v[1] = y1;
    v[2] = y2;
    v[3] = y3;
    v[4] = y4;
    v[5] = y5;
    v[6] = y6;
}

// Forward transforms (exp(-2 pi i ...)) of the workgroup, unscaled; registers as
// FftLane before and after.  buf: blockDim.x * FE entries, free to overwrite once
// every thread has arrived.  tw[k] = exp(-2 pi i k / P), k < P/2.  The
// inverse of x is the forward transform with real and imaginary parts exchanged
// before and after.
template <bool IL, bool SMALL>
__device__ __forceinline__ void fft_fwd(double2 (&v)[FE], const FftLane<IL, SMALL>& L, double2* buf,
                                        const double2* __restrict__ tw) {
    const int logP = L.logP;
    if constexpr (SMALL) {
        if (logP == 1) {
#pragma unroll
            for (int q = 0; q < 4; ++q) dft2(v[q], v[q + 4]);
        } else {
#pragma unroll
            for (int q = 0; q < 2; ++q) dft4(v[q], v[q + 2], v[q + 4], v[q + 6]);
        }
        return;
    }
    dft8(v);
    for (int lN = 3; lN < logP; lN += 3) {   // lN: log2 of the length of the sub-transforms done
        const int rem = logP - lN;
        // the next pass's twiddles, on their way during the exchange: w, w^2 and w^4
        // of the radix-8 butterfly; of a last pass of radix 2 or 4, whose
        // butterfly q holds registers q + r FE / R and stays in place, those of
        // the four or (w and w^2) two butterflies
        int iw[4];
        if (rem >= 3) {
            iw[0] = (L.t & ((1 << lN) - 1)) << (rem - 3);
            iw[1] = 2 * iw[0];
            iw[2] = 4 * iw[0];
            iw[3] = 0;
        } else {
            iw[0] = L.pos(0);
            iw[1] = L.pos(1);
            iw[2] = rem == 1 ? L.pos(2) : 2 * iw[0];
            iw[3] = rem == 1 ? L.pos(3) : 2 * iw[1];
        }
        double2 w[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] = tw[iw[q]];
        const int s = lN - 3;   // the pass just done: sub-transforms 2^s -> 2^lN
        const int base = ((L.t >> s) << lN) + (L.t & ((1 << s) - 1));
        __syncthreads();
#pragma unroll
        for (int k = 0; k < FE; ++k) buf[L.slot(base + (k << s), L.c)] = v[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < FE; ++k) v[k] = buf[L.slot(L.pos(k), L.c)];
        if (rem >= 3) {
            const double2 w3 = cmul(w[0], w[1]);
            v[1] = cmul(v[1], w[0]);
            v[2] = cmul(v[2], w[1]);
            v[3] = cmul(v[3], w3);
            v[4] = cmul(v[4], w[2]);
            v[5] = cmul(v[5], cmul(w[0], w[2]));
            v[6] = cmul(v[6], cmul(w[1], w[2]));
            v[7] = cmul(v[7], cmul(w3, w[2]));
            dft8(v);
        } else if (rem == 1) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v[q + 4] = cmul(v[q + 4], w[q]);
                dft2(v[q], v[q + 4]);
            }
        } else {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                v[q + 2] = cmul(v[q + 2], w[q]);
                v[q + 4] = cmul(v[q + 4], w[q + 2]);
                v[q + 6] = cmul(v[q + 6], cmul(w[q], w[q + 2]));
                dft4(v[q], v[q + 2], v[q + 4], v[q + 6]);
            }
        }
    }
}

template <bool SMALL, class T>
__device__ __forceinline__ void rows_fwd_body(const FFTPlan& F, const T* __restrict__ g, double2* buf, int bx) {
    const FftLane<false, SMALL> L(F.logP);
    const int pair0 = bx << L.lc, half = F.P / 2;
    double2 v[FE];
#pragma unroll
    for (int k = 0; k < FE; ++k) {
        const int n = L.pos(k), r0 = 2 * (pair0 + L.col(k));
        v[k] = make_double2(0.0, 0.0);
        if (k >= L.LOWER) continue;
        const bool in0 = n < F.cols && r0 < F.rows, in1 = in0 && r0 + 1 < F.rows;
        const T re = g[in0 ? (size_t)r0 * F.cols + n : 0];   // (loaded in any case: no branch)
        const T im = g[in1 ? (size_t)(r0 + 1) * F.cols + n : 0];
        if (in0) v[k].x = re;
        if (in1) v[k].y = im;
    }
    fft_fwd(v, L, buf, F.tw);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < FE; ++k) buf[L.slot(L.pos(k), L.col(k))] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < FE; ++k) {
        const int u = L.pos(k), r0 = 2 * (pair0 + L.col(k));
        if (k > L.LOWER || u > half || r0 >= F.rows) continue;
        const double2 Z = v[k];
        const double2 W = buf[L.slot((F.P - u) & (F.P - 1), L.col(k))];   // Z(-u); conj taken below
        // X0 = (Z + conj W) / 2 ;  X1 = (Z - conj W) / (2i)
        F.S[(size_t)r0 * F.SP + u] = make_double2(0.5 * (Z.x + W.x), 0.5 * (Z.y - W.y));
        if (r0 + 1 < F.rows)
            F.S[(size_t)(r0 + 1) * F.SP + u] = make_double2(0.5 * (Z.y + W.y), -0.5 * (Z.x - W.x));
    }
}

template <bool SMALL, class T>
__global__ __launch_bounds__(512) void k_rows_fwd(FFTPlan F, const T* __restrict__ g, const int* __restrict__ run,
                                                  const int* __restrict__ halt) {
    if (halt && *halt) return;
    if (run && !*run) return;
    extern __shared__ double2 buf[];
    rows_fwd_body<SMALL>(F, g, buf, blockIdx.x);
}

// h(w) of eq. (3.2) from w^2 <= 2 pi^2.  The square root by Goldschmidt's
// iteration from the hardware's estimate; cos w = 2 cos^2(w / 2) - 1 by the
// Taylor series in (w / 2)^2 <= 4.94, whose 15th term is below 2e-20: about 30
// instructions where the library's range reduction for any argument took most
// of the column kernel's arithmetic (all three
// kernels, 2048^2: 206 -> 152 us, 512^2: 27.6 -> 25.7).  Its error against 128 bits
// is that of sqrt and cos called: 5e-16 at rho = 0.8, 2e-15 towards rho = 1/2.
__device__ __forceinline__ double window_h(double w2, double mu, double rho) {
    const double x = w2 + 1e-300;   // (finite estimate at the origin)
    double y = __builtin_amdgcn_rsq(x);
    double g = x * y, hy = 0.5 * y;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const double r = fma(-hy, g, 0.5);
        g = fma(g, r, g);
        hy = fma(hy, r, hy);
    }
    const double w = fma(fma(-g, g, x), hy, g);
    const double q = 0.25 * w2;
    double c = 1.0 / 304888344611713860501504000000.0;   // 1 / 28!
    constexpr double f[13] = {1.0 / 403291461126605635584000000.0, 1.0 / 620448401733239439360000.0,
                              1.0 / 1124000727777607680000.0, 1.0 / 2432902008176640000.0,
                              1.0 / 6402373705728000.0, 1.0 / 20922789888000.0, 1.0 / 87178291200.0,
                              1.0 / 479001600.0, 1.0 / 3628800.0, 1.0 / 40320.0, 1.0 / 720.0, 1.0 / 24.0, 0.5};
#pragma unroll
    for (int i = 0; i < 13; ++i) c = fma(-q, c, f[i]);   // alternating: 1/26! - q/28!, ...
    c = fma(-q, c, 1.0);
    const double cw = fma(2.0 * c, c, -1.0);
    return (w + mu) * fma(1.0 - rho, cw, rho);
}

template <bool SMALL>
__device__ __forceinline__ void cols_body(const FFTPlan& F, double mu, double rho, double2* buf, int bx) {
    const FftLane<true, SMALL> L(F.logP);
    const int u0 = bx << L.lc;
    double2 v[FE];
#pragma unroll
    for (int k = 0; k < FE; ++k) {
        const int r = L.pos(k), u = u0 + L.col(k);
        const bool in = r < F.rows && u < F.SP;
        v[k] = make_double2(0.0, 0.0);
        if (k >= L.LOWER) continue;
        const double2 x = F.S[in ? (size_t)r * F.SP + u : 0];   // (loaded in any case: no branch)
        if (in) v[k] = x;
    }
    fft_fwd(v, L, buf, F.tw);
    const double two_pi_over_P = 6.283185307179586 / (double)F.P;
#pragma unroll
    for (int k = 0; k < FE; ++k) {
        const int q = L.pos(k), u = u0 + L.col(k);
        const int vv = q < F.P / 2 ? q : q - F.P;
        const double wu = two_pi_over_P * (double)u, wv = two_pi_over_P * (double)vv;
        const double h = window_h(fma(wv, wv, wu * wu), mu, rho);
        v[k] = make_double2(v[k].y * h, v[k].x * h);   // exchanged for the inverse
        if (k & 1) __builtin_amdgcn_sched_barrier(0);   // (two windows at a time: registers)
    }
    fft_fwd(v, L, buf, F.tw);
#pragma unroll
    for (int k = 0; k < FE; ++k) {
        const int r = L.pos(k), u = u0 + L.col(k);
        if (k < L.LOWER && r < F.rows && u < F.SP) F.S[(size_t)r * F.SP + u] = make_double2(v[k].y, v[k].x);
    }
}

template <bool SMALL>
__global__ __launch_bounds__(512) void k_cols(FFTPlan F, double mu, double rho, const int* __restrict__ run,
                                              const int* __restrict__ halt) {
    if (halt && *halt) return;
    if (run && !*run) return;
    extern __shared__ double2 buf[];
    // neighbouring columns on one XCD: they share cache lines of S
    const int per = gridDim.x / 8, b = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (b * F.NF < F.SP) cols_body<SMALL>(F, mu, rho, buf, b);
}

// T: the type of z (float32 results are rounded once).  With xp, z is also
// written to R's padded float64 copies (xp row-major with row pitch pitchX, xTp
// transposed with pitch pitchXT, both PAD-offset), as R's prep would write them.
template <bool SMALL, class T>
__device__ __forceinline__ void rows_inv_body(const FFTPlan& F, T* __restrict__ z, double2* buf, int bx,
                                              double* __restrict__ xp = nullptr,
                                              double* __restrict__ xTp = nullptr, int pitchX = 0,
                                              int pitchXT = 0) {
    const FftLane<false, SMALL> L(F.logP);
    const int pair0 = bx << L.lc, half = F.P / 2;
    double2 v[FE];
#pragma unroll
    for (int k = 0; k < FE; ++k) {
        const int p = L.pos(k), r0 = 2 * (pair0 + L.col(k));
        const int u = p <= half ? p : F.P - p;
        const bool in0 = r0 < F.rows, in1 = r0 + 1 < F.rows;   // (loaded in any case: no branch)
        double2 X0 = F.S[in0 ? (size_t)r0 * F.SP + u : 0], X1 = F.S[in1 ? (size_t)(r0 + 1) * F.SP + u : 0];
        if (!in0) X0 = make_double2(0.0, 0.0);
        if (!in1) X1 = make_double2(0.0, 0.0);
        if (p > half) X0.y = -X0.y, X1.y = -X1.y;
        v[k] = make_double2(X0.y + X1.x, X0.x - X1.y);   // X0 + i X1, exchanged for the inverse
    }
    fft_fwd(v, L, buf, F.tw);
    const double scale = 1.0 / ((double)F.P * (double)F.P);
#pragma unroll
    for (int k = 0; k < FE; ++k) {
        const int j = L.pos(k), r0 = 2 * (pair0 + L.col(k));
        if (k >= L.LOWER || j >= F.cols || r0 >= F.rows) continue;
        const double a = v[k].y * scale, b = v[k].x * scale;
        z[(size_t)r0 * F.cols + j] = (T)a;
        if (xp) {
            xp[(size_t)r0 * pitchX + PAD + j] = a;
            xTp[(size_t)j * pitchXT + PAD + r0] = a;
        }
        if (r0 + 1 < F.rows) {
            z[(size_t)(r0 + 1) * F.cols + j] = (T)b;
            if (xp) {
                xp[(size_t)(r0 + 1) * pitchX + PAD + j] = b;
                xTp[(size_t)j * pitchXT + PAD + r0 + 1] = b;
            }
        }
    }
}

template <bool SMALL, class T>
__global__ __launch_bounds__(512) void k_rows_inv(FFTPlan F, T* __restrict__ z, const int* __restrict__ run,
                                                  const int* __restrict__ halt,
                                                  double* __restrict__ xp, double* __restrict__ xTp,
                                                  int pitchX, int pitchXT) {
    if (halt && *halt) return;
    if (run && !*run) return;
    extern __shared__ double2 buf[];
    rows_inv_body<SMALL>(F, z, buf, blockIdx.x, xp, xTp, pitchX, pitchXT);
}

// Batched: z = M g per slice (of each form its slices).
template <bool SMALL>
__global__ __launch_bounds__(512) void kb_rows_fwd(const SliceDev* __restrict__ sl, ItemTable t) {
    extern __shared__ double2 buf[];
    for_items(t, [&](int s, int lin) {
        const SliceDev& S = sl[s];
        if ((S.F.logP < 3) != SMALL || gmem(S.sc)->halt) return;
        FFTPlan F = S.F;
        F.S = gmem(F.S);
        F.tw = cmem(F.tw);
        rows_fwd_body<SMALL>(F, (const double*)gmem(S.g), buf, lin);
    });
}

template <bool SMALL>
__global__ __launch_bounds__(512, 4) void kb_cols(const SliceDev* __restrict__ sl, ItemTable t, double mu,
                                               double rho) {
    extern __shared__ double2 buf[];
    for_items(t, [&](int s, int lin) {
        const SliceDev& S = sl[s];
        if ((S.F.logP < 3) != SMALL || gmem(S.sc)->halt) return;
        FFTPlan F = S.F;
        F.S = gmem(F.S);
        F.tw = cmem(F.tw);
        cols_body<SMALL>(F, mu, rho, buf, lin);
    });
}

template <bool SMALL>
__global__ __launch_bounds__(512) void kb_rows_inv(const SliceDev* __restrict__ sl, ItemTable t) {
    extern __shared__ double2 buf[];
    for_items(t, [&](int s, int lin) {
        const SliceDev& S = sl[s];
        if ((S.F.logP < 3) != SMALL || gmem(S.sc)->halt) return;
        FFTPlan F = S.F;
        F.S = gmem(F.S);
        F.tw = cmem(F.tw);
        rows_inv_body<SMALL>(F, (double*)gmem(S.z), buf, lin);
    });
}

// Threads of a workgroup: one transform, at least a wave.  (Two columns side by
// side read 32 consecutive bytes, but 700^2 took 60 us so and 50 one by one: the
// neighbours' lines come from the XCD's L2.  A batch's workgroups have one size.)
int fft_threads(int P) { return std::max(64, P / FE); }
// Transforms of a workgroup of `threads`, which must hold at least one.
int fft_per_group(int P, int threads) { return threads * FE / P; }

template <bool SMALL>
void launch_precond_b_form(hipStream_t st, const SliceDev* sl, ItemTable rows, ItemTable cols, int threads,
                           double mu, double rho) {
    const size_t lds = (size_t)threads * FE * sizeof(double2);
    hipLaunchKernelGGL(kb_rows_fwd<SMALL>, dim3(rows.grid), dim3(threads), lds, st, sl, rows);
    hipLaunchKernelGGL(kb_cols<SMALL>, dim3(cols.grid), dim3(threads), lds, st, sl, cols, mu, rho);
    hipLaunchKernelGGL(kb_rows_inv<SMALL>, dim3(rows.grid), dim3(threads), lds, st, sl, rows);
}

void launch_precond_b(hipStream_t st, const SliceDev* sl, ItemTable rows, ItemTable cols, int threads, int forms,
                      double mu, double rho) {
    if (forms & FFT_FORM_SMALL) launch_precond_b_form<true>(st, sl, rows, cols, threads, mu, rho);
    if (forms & FFT_FORM_LARGE) launch_precond_b_form<false>(st, sl, rows, cols, threads, mu, rho);
}

template <bool SMALL, class T>
void launch_precond_form(hipStream_t st, const FFTPlan& F, double mu, double rho, const T* g, T* z,
                         const int* halt, const int* run, const GeomDev* G, double* xp, double* xTp) {
    const int nt = fft_threads(F.P), nrow = ((F.rows + 1) / 2 + F.NF - 1) / F.NF;
    const size_t lds = (size_t)nt * FE * sizeof(double2);
    hipLaunchKernelGGL((k_rows_fwd<SMALL, T>), dim3(nrow), dim3(nt), lds, st, F, g, run, halt);
    const int ncb = (F.SP + F.NF - 1) / F.NF;
    hipLaunchKernelGGL(k_cols<SMALL>, dim3((ncb + 7) / 8 * 8), dim3(nt), lds, st, F, mu, rho, run, halt);
    hipLaunchKernelGGL((k_rows_inv<SMALL, T>), dim3(nrow), dim3(nt), lds, st, F, z, run, halt,
                       G ? xp : nullptr, G ? xTp : nullptr, G ? G->pitchX : 0, G ? G->pitchXT : 0);
}

template <class T>
void launch_precond_t(hipStream_t st, const FFTPlan& F, double mu, double rho, const T* g, T* z,
                      const int* halt, const int* run, const GeomDev* G, double* xp, double* xTp) {
    if (fft_form(F) == FFT_FORM_SMALL) launch_precond_form<true>(st, F, mu, rho, g, z, halt, run, G, xp, xTp);
    else launch_precond_form<false>(st, F, mu, rho, g, z, halt, run, G, xp, xTp);
}

void launch_precond(hipStream_t st, const FFTPlan& F, double mu, double rho, const float* g, float* z,
                    const int* halt, const int* run) {
    launch_precond_t(st, F, mu, rho, g, z, halt, run, nullptr, nullptr, nullptr);
}
void launch_precond(hipStream_t st, const FFTPlan& F, double mu, double rho, const double* g, double* z,
                    const int* halt, const int* run, const GeomDev* G, double* xp, double* xTp) {
    launch_precond_t(st, F, mu, rho, g, z, halt, run, G, xp, xTp);
}

}  // namespace sp
