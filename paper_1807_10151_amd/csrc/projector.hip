// Matrix-free parallel-beam projector R (ray-driven gather) and its exact
// transpose R^T (pixel-driven gather, no atomics).
//
// R[(a,k),(i,j)] is the length of ray (a,k) inside pixel (i,j) (the projection
// matrix of Section 2, rays as in Section 4.1).  R^T evaluates each weight as
// the chord length of a line through a square (offset d = s_k - t of the bin
// from the projection t of the pixel centre, the clamped trapezoid u of
// chord_u, times the angle's wmax).  R walks each ray band by band and splits
// a band's path length at the pixel boundary it crosses (ray_split): the same
// lengths in exact arithmetic, equal to rounding in float64, so R^T is the
// adjoint of R to float64 rounding (axis-parallel angles use the trapezoid in
// both, bit for bit, with its half weight for a ray on a pixel edge).  Data
// are float32; coordinates, weights and sums are float64 (FP64 FMA issues at
// the non-packed FP32 rate on CDNA4, and float32 angles alone would move a ray
// by ~1e-5 pixel at radius 256).
//
// Gathers stay inside one zero-padded row (of the image copy, its transpose or
// the sinogram).  R^T reads through buffer loads whose descriptor spans the
// row, so an index past either end reads 0 in hardware; R clamps its index
// into the row's pads.  A legitimate candidate always lies inside the row (its
// pads included), which the host index checker verifies for every geometry it
// is given.
//
// Forward walk.  For a vertical angle a ray crosses every image row; within
// row i it meets at most two pixels, as its crossing point moves by `slope`
// (|slope| <= 1) columns per row.  A lane owns one ray and the 64 lanes of a
// wave walk the union of their (nonempty) row ranges together, so each step
// gathers neighbouring addresses of one row.  R's wave table (WaveDev) gives
// each wave its rays: 16 consecutive bins of four neighbouring angles (rays
// whose image extents differ little, so few lane-steps fall outside a lane's
// own ray), the last nB % 16 bins of consecutive angles of one class packed
// into full waves, or 64 bins of one axis-parallel angle; a workgroup's four
// waves are four consecutive table entries (the four 16-bin parts of one
// 64-bin chunk of the same angles), and the workgroups run in a
// host-computed order (project_order).  Horizontal angles walk columns of a zero-padded
// transposed copy.  R of a float32 image (the standalone operators') gives
// a lane two neighbouring rays where the bin spacing allows it (ray_pair); the
// solvers' float64 vectors keep one.
//
// Backward gather.  A lane owns PX (2 or 4) pixels of one row, 8 columns
// apart, and loops over the angles, which are sorted into four classes
// (vertical/horizontal x oblique/axis-parallel) so the inner loop has no
// branch; at each angle a pixel's nonzero bins are the NB bins from padded
// index trunc(kf), read from a zero-padded sinogram (float32, or float64 for
// the solvers' residual) whose rows carry the angle's wmax.
#include "sp_internal.h"
#include "sp_reduce.h"
#include "sp_scalar.h"
#include "sp_walk.h"

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

namespace sp {

// 32 x 32 tile (bx, by): padded copy and padded transposed copy of a float32
// image (float32 copies for the two-ray form, else float64) or of a float64
// iterate.
template <class T, class C>
__device__ __forceinline__ void prep_body(const GeomDev& G, const T* __restrict__ x,
                                          C* __restrict__ xp, C* __restrict__ xTp, int bx,
                                          int by) {
    __shared__ T tile[32][33];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int j = bx * 32 + tx;
#pragma unroll
    for (int r = 0; r < 32; r += 8) {
        const int i = by * 32 + ty + r;
        T v = 0;
        if (i < G.rows && j < G.cols) {
            v = x[(size_t)i * G.cols + j];
            xp[(size_t)i * G.pitchX + PAD + j] = (C)v;
        }
        tile[ty + r][tx] = v;
    }
    __syncthreads();
    const int ii = by * 32 + tx;
#pragma unroll
    for (int r = 0; r < 32; r += 8) {
        const int jj = bx * 32 + ty + r;
        if (ii < G.rows && jj < G.cols)
            xTp[(size_t)jj * G.pitchXT + PAD + ii] = (C)tile[tx][ty + r];
    }
}

template <class T, class C>
__global__ __launch_bounds__(256) void k_prep(GeomDev G, const T* __restrict__ x,
                                              C* __restrict__ xp, C* __restrict__ xTp,
                                              const int* __restrict__ halt) {
    if (halt && *halt) return;
    prep_body(G, x, xp, xTp, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(256) void kb_prep(const SliceDev* __restrict__ sl, ItemTable t, int which) {
    for_items(t, [&](int s, int lin) {
        const SliceDev& S = sl[s];
        if (gmem(S.sc)->halt) return;
        const GeomDev G = S.G;
        const int gx = (G.cols + 31) / 32;
        prep_body(G, (const double*)batch_vec(S, which), gmem(S.xp), gmem(S.xTp), lin % gx, lin / gx);
    });
}

void launch_prep_b(hipStream_t st, const SliceDev* sl, ItemTable t, int which) {
    hipLaunchKernelGGL(kb_prep, dim3(t.grid), dim3(256), 0, st, sl, t, which);
}

void launch_prep(hipStream_t st, const GeomDev& G, const float* x, double* xp, double* xTp,
                 const int* halt) {
    dim3 grid((G.cols + 31) / 32, (G.rows + 31) / 32);
    hipLaunchKernelGGL((k_prep<float, double>), grid, dim3(256), 0, st, G, x, xp, xTp, halt);
}

void launch_prep(hipStream_t st, const GeomDev& G, const double* x, double* xp, double* xTp,
                 const int* halt) {
    dim3 grid((G.cols + 31) / 32, (G.rows + 31) / 32);
    hipLaunchKernelGGL((k_prep<double, double>), grid, dim3(256), 0, st, G, x, xp, xTp, halt);
}

void launch_prep32(hipStream_t st, const GeomDev& G, const float* x, float* zp, float* zTp,
                   const int* halt) {
    dim3 grid((G.cols + 31) / 32, (G.rows + 31) / 32);
    hipLaunchKernelGGL((k_prep<float, float>), grid, dim3(256), 0, st, G, x, zp, zTp, halt);
}

__device__ __forceinline__ int wave_min(int v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = min(v, __shfl_xor(v, off, 64));
    return v;
}
__device__ __forceinline__ int wave_max(int v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = max(v, __shfl_xor(v, off, 64));
    return v;
}

// ---- range-checked row gathers ---------------------------------------------
typedef double d2v __attribute__((ext_vector_type(2)));
typedef float f2v __attribute__((ext_vector_type(2)));
typedef float f4v __attribute__((ext_vector_type(4)));
// Descriptor word 3 of a raw gfx9 buffer (32-bit data format, no swizzle).
constexpr int BUF_WORD3 = 0x00020000;

// Buffer resource over `bytes` bytes from `row` (wave-uniform).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void* row, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(row), (short)0, bytes, BUF_WORD3);
}

// The N elements e, e + 1, ... of a row; every element past either end of the
// row reads 0 (e is taken as unsigned, so a negative index is past the end).
template <class T, int N>
__device__ __forceinline__ void row_load(__amdgpu_buffer_rsrc_t r, unsigned e, T (&v)[N]) {
    const unsigned off = e * (unsigned)sizeof(T);
    if constexpr (sizeof(T) == 8 && N == 2) {
        const d2v t = __builtin_bit_cast(d2v, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
        v[0] = t.x;
        v[1] = t.y;
    } else if constexpr (sizeof(T) == 4 && N == 2) {
        const f2v t = __builtin_bit_cast(f2v, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
        v[0] = t.x;
        v[1] = t.y;
    } else if constexpr (sizeof(T) == 4 && N == 4) {
        const f4v t = __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
        v[0] = t.x;
        v[1] = t.y;
        v[2] = t.z;
        v[3] = t.w;
    } else {
#pragma unroll
        for (int q = 0; q < N; ++q) {
            if constexpr (sizeof(T) == 8)
                v[q] = __builtin_bit_cast(
                    double, __builtin_amdgcn_raw_buffer_load_b64(r, off + 8u * q, 0, 0));
            else
                v[q] = __builtin_bit_cast(
                    float, __builtin_amdgcn_raw_buffer_load_b32(r, off + 4u * q, 0, 0));
        }
    }
}

// The forward walks gather with plain global loads from a row, the index
// clamped to the row's last full window: a clamped index lands in the row's
// zero pads, and every true candidate of such a step lies outside the image.
// (Buffer loads, whose descriptor is rebuilt per row on the scalar unit,
// measured 3-4% slower here; the backprojector, one row per angle, gains.)
struct RowRef {
    const char* p;
    int bytes;
};
__device__ __forceinline__ RowRef row_ref(const void* row, int bytes) {
    return RowRef{reinterpret_cast<const char*>(row), bytes};
}
template <class T, int N>
__device__ __forceinline__ void row_load(RowRef r, unsigned e, T (&v)[N]) {
    const unsigned emax = (unsigned)(r.bytes / (int)sizeof(T) - N);
    e = min(e, emax);
    const T* q = reinterpret_cast<const T*>(r.p) + e;
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = q[i];
}
// ---- forward walk ----------------------------------------------------------
// The wave's common step range [lo, hi) from the lanes' own ranges: lanes
// without a ray, or whose ray misses the image, take no part.
__device__ __forceinline__ void wave_range(int l, int h, bool valid, int nmaj, int& lo, int& hi) {
    if (!valid || l >= h) {
        l = nmaj;
        h = 0;
    }
    lo = __builtin_amdgcn_readfirstlane(wave_min(l));
    hi = __builtin_amdgcn_readfirstlane(wave_max(h));
}

// One axis-parallel ray's sum over the steps [lo, hi), with the
// trapezoid per candidate (its half weight for a ray on a pixel edge).
// HORIZ = walk columns of the transposed copy.  img points at element PAD of
// row 0 of the padded copy.  Candidate q of step m is minor index
// floor(nf_m) + 1 + q; nf carries the + 1 + PAD of the padded index, so the
// first candidate's padded index is trunc(nf) where nf >= 0 (a negative nf
// reads past the row's start, i.e. 0, as does any index past its end; every
// true candidate of such a step lies outside the image).  The minor coordinate
// of candidate q is taken from the index read -- (o + q - PAD) - xoff for
// columns, yoff - (o + q - PAD) for rows, exact small half-integers.
// Axis-parallel rays cross the whole image, so their waves are among the
// longest of the launch: U steps per iteration keep U gathers in flight, as a
// wave's walk is otherwise bound by the latency of its chain of gathers.
template <bool HORIZ, class T>
__device__ __forceinline__ double ray_sum_axis(const GeomDev& G, const AngleDev& A, double sk,
                                               const T* __restrict__ img, int lo, int hi) {
    constexpr int NC = 2, U = 4;
    const int pitch = HORIZ ? G.pitchXT : G.pitchX;
    double acc = 0.0;
    const double start = walk_start<HORIZ>(G, A, sk);
    const double fm = HORIZ ? A.s : A.c;   // factor of the per-candidate fma
    const double c2 = HORIZ ? G.yoff + (double)PAD : -(double)PAD - G.xoff;
    const double fM = HORIZ ? A.c : A.s;   // factor of the shared (major) product
    const double dM = HORIZ ? 1.0 : -1.0;  // major coordinate step
    double cM = HORIZ ? (double)lo - G.xoff : G.yoff - (double)lo;
    double nf = fma((double)lo, A.slope, start + (double)(1 + PAD));
    const int rowbytes = pitch * (int)sizeof(T);
    const char* rowp = reinterpret_cast<const char*>(img - PAD) + (size_t)lo * rowbytes;
    auto step = [&](const T (&v)[NC], int o, double cMv) {
        const double P = cMv * fM;
        const double cm0 = HORIZ ? c2 - (double)o : (double)o + c2;
#pragma unroll
        for (int q = 0; q < NC; ++q) {
            const double cm = HORIZ ? cm0 - (double)q : cm0 + (double)q;
            const double d = sk - fma(cm, fm, P);
            acc = fma(chord_u<true>(d, A.einv, A.inv), (double)v[q], acc);
        }
    };
    int m = lo;
    for (; m + U <= hi; m += U) {
        int o[U];
        T v[U][NC];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            o[u] = (int)nf;
            row_load<T, NC>(row_ref(rowp + u * rowbytes, rowbytes), (unsigned)o[u], v[u]);
            nf += A.slope;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            step(v[u], o[u], cM);
            cM += dM;
        }
        rowp += U * rowbytes;
    }
    for (; m < hi; ++m) {
        const int o = (int)nf;
        T v[NC];
        row_load<T, NC>(row_ref(rowp, rowbytes), (unsigned)o, v);
        step(v, o, cM);
        nf += A.slope;
        cM += dM;
        rowp += rowbytes;
    }
    return acc;
}

// One oblique ray's sum of u-weighted values over the steps [lo, hi), by
// splitting each major step's band at the pixel boundary.  With |slope| <= 1
// the ray crosses a band (an image row for vertical angles, a column of the
// transposed copy for horizontal ones) over a minor-axis interval of length
// |slope| starting at lp = b0 + m * slope (padded minor coordinate, pixel q
// spanning [q, q + 1)), so it meets at most pixels floor(lp) and
// floor(lp) + 1.  The share of the band's path length (wmax, applied by the
// caller) in the first is f = clamp((floor(lp) + 1 - lp) / |slope|, 0, 1) =
// clamp((1 - fract(lp)) / |slope|, 0, 1) and the rest falls in the second:
// the exact chord lengths of the pixel model, the same values chord_u * wmax
// gives up to rounding.  lp advances by slope per step (its rounding error
// stays ~1e-11 pixel over the longest walk).  A truncated index below the row
// or past it reads 0, where the pixels contribute 0.  The longest waves set
// the launch's length and their walk is bound by the latency of its chain of
// gathers, so U steps' gathers are issued before their math.
template <bool HORIZ, class T>
__device__ __forceinline__ double ray_split(const GeomDev& G, const AngleDev& A, double sk,
                                            const T* __restrict__ img, int lo, int hi) {
    const int pitch = HORIZ ? G.pitchXT : G.pitchX;
    double acc = 0.0;
    constexpr int U = 2;   // steps per iteration: their gathers are in flight together
    const double sig = A.slope;
    const double isg = 1.0 / fabs(sig);
    double lp = fma((double)lo, sig, split_b0<HORIZ>(G, A, sk));
    const int rowbytes = pitch * (int)sizeof(T);
    const char* rowp = reinterpret_cast<const char*>(img - PAD) + (size_t)lo * rowbytes;
    auto step = [&](const T (&v)[2], double lpv) {
        const double v0 = v[0], v1 = v[1];
        const double f = fmin(fmax(fma(__builtin_amdgcn_fract(lpv), -isg, isg), 0.0), 1.0);
        acc += fma(f, v0 - v1, v1);
    };
    int m = lo;
    for (; m + U <= hi; m += U) {
        double lpu[U];
        T v[U][2];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            lpu[u] = lp;
            row_load<T, 2>(row_ref(rowp + u * rowbytes, rowbytes), (unsigned)(int)lp, v[u]);
            lp += sig;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) step(v[u], lpu[u]);
        rowp += U * rowbytes;
    }
    for (; m < hi; ++m) {
        T v[2];
        row_load<T, 2>(row_ref(rowp, rowbytes), (unsigned)(int)lp, v);
        step(v, lp);
        lp += sig;
        rowp += rowbytes;
    }
    return acc;
}

// Two neighbouring oblique rays of one angle from a float32 image over the steps
// [lo, hi): acc[0] the one with the smaller minor coordinate.  From about unit
// bin spacing up the two rays' bands are 1 to 2 pixels apart (pair_fits), so
// the four pixels j .. j + 3 that one 16-byte gather brings serve both, where
// ray_split gathers 16 bytes per ray and band and the vector L1 paces it.
// Bound: the L1's return path (about 23 cycles per gather; 0.87 busy at
// 1024^2) with the float64 VALU (0.82) beside it, 10.5 instructions per ray
// and band.  Range-checked buffer loads save the index clamp and the 64-bit
// address (2-9%).  Four bands per iteration (512^2: two 102, three 93, four
// 88 us) with four waves per SIMD; half as many waves as one ray per lane.
// R with its copies: 512^2 x 720 98 -> 88 us, 724^2 x 1016 273 -> 188, 1024^2 x
// 1432 644 -> 436, 2048^2 x 2048 3.52 -> 2.31 ms (uniform random image).
template <bool HORIZ>
__device__ __forceinline__ void ray_pair(const GeomDev& G, const AngleDev& A, double sk,
                                         const float* __restrict__ img, int lo, int hi, double (&acc)[2]) {
    const int pitch = HORIZ ? G.pitchXT : G.pitchX;
    constexpr int U = 4;   // bands per iteration
    const double sig = A.slope;
    const double isg = 1.0 / fabs(sig), delta = pair_delta(G, A);
    double lp = fma((double)lo, sig, split_b0<HORIZ>(G, A, sk));
    const int rowbytes = pitch * 4;
    const char* rowp = reinterpret_cast<const char*>(img - PAD) + (size_t)lo * rowbytes;
    acc[0] = acc[1] = 0.0;
    auto step = [&](const float (&v)[4], double lpv) {
        double f, g1, g2;
        pair_shares(__builtin_amdgcn_fract(lpv), isg, delta, f, g1, g2);
        const double v0 = v[0], v1 = v[1], v2 = v[2], v3 = v[3];
        const double d12 = v1 - v2;
        acc[0] += fma(f, v0 - v1, v1);
        acc[1] += fma(g1, d12, fma(g2, v2 - v3, v3));
    };
    int m = lo;
    for (; m + U <= hi; m += U) {
        double lpu[U];
        float v[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            lpu[u] = lp;
            row_load<float, 4>(row_rsrc(rowp + u * rowbytes, rowbytes), (unsigned)(int)lp, v[u]);
            lp += sig;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) step(v[u], lpu[u]);
        rowp += U * rowbytes;
    }
    for (; m < hi; ++m) {
        float v[4];
        row_load<float, 4>(row_rsrc(rowp, rowbytes), (unsigned)(int)lp, v);
        step(v, lp);
        lp += sig;
        rowp += rowbytes;
    }
}

// Stores ray (row a, bin k): v = (R x)_{a,k}, or the residual r = R x - b when
// o.b != nullptr.  The value goes, rounded to float32, to o.out[a*nB + k]; the
// padded sinogram that feeds R^T gets it times the angle's wmax (see bp_class)
// unrounded in o.outpd[a*pitchB + PAD + k]; o.wout receives v unrounded at
// a*nB + k (each nullable).  Returns the ray's term of the workgroup's float64
// partial: r^2, or with dq (and no b) v dq[a*nB + k].
__device__ __forceinline__ double project_value(const GeomDev& G, int a, double wmax, int k,
                                                bool valid, double acc, const RayOut& o) {
    double r2 = 0.0;
    if (valid) {
        double v;
        const size_t i = (size_t)a * G.nB + k;
        if (o.b) {
            v = fma(acc, G.pixel, -(double)o.b[i]);
            r2 = v * v;
        } else {
            v = acc * G.pixel;
            if (o.dq) r2 = v * o.dq[i];
        }
        if (o.out) o.out[i] = (float)v;
        if (o.wout) o.wout[i] = v;
        if (o.outpd) o.outpd[(size_t)a * G.pitchB + PAD + k] = v * wmax;
    }
    return r2;
}
// The workgroup's partial (its first 256 threads; the others have ended).
__device__ __forceinline__ void project_partial(double r2, const RayOut& o, int pidx) {
    __shared__ double red[4];
    if (!o.b && !o.dq) return;
    const double tot = block_sum(r2, red);
    if (threadIdx.x == 0) o.partials[pidx] = tot;
}

// The rays of one lane of R, and the wave's common step range.  T: the type of
// the padded copies, and with it the form: one ray from float64 copies, two
// neighbouring ones, k and k + 1, from float32 ones (one for axis-parallel
// angles).
template <class T>
struct LaneRays {
    static constexpr bool PAIR = sizeof(T) == 4;
    AngleDev A;
    int ai, k, flags, lo, hi;
    bool valid, valid2;
    double s0, s1;

    // Entry wi of the form's wave table of nw entries (lane l one or two of its
    // rays, see WaveDev).
    __device__ __forceinline__ void set(const GeomDev& G, const AngleDev* __restrict__ ang,
                                        const WaveDev* __restrict__ waves, int wi, int nw) {
        const bool wvalid = wi < nw;
        const WaveDev W = waves[wvalid ? wi : 0];
        flags = ang[W.a0].flags;   // the wave's class (wave-uniform)
        const bool two = PAIR && !(flags & ANG_AXIS);
        valid = wvalid && (two ? wave_pair(W, threadIdx.x & 63, G.nB, ai, k)
                               : wave_ray(W, threadIdx.x & 63, G.nB, ai, k));
        if (!valid) {   // no ray: a valid angle of the wave's class, summing nothing
            ai = W.a0;
            k = 0;
        }
        valid2 = two && valid && k + 1 < G.nB;
        A = ang[ai];
        s0 = bin_pos((double)k, G);
        s1 = bin_pos((double)(k + 1), G);
        int l, h;
        auto steps = [&](double s, int& a, int& b) {
            if (flags & ANG_HORIZ) ray_steps<true>(G, A, s, a, b);
            else ray_steps<false>(G, A, s, a, b);
        };
        steps(s0, l, h);
        if (PAIR && valid2) {   // the union of the two rays' nonempty ranges
            int l1, h1;
            steps(s1, l1, h1);
            if (l1 < h1) {
                h = l < h ? max(h, h1) : h1;
                l = l < h ? min(l, l1) : l1;
            }
        }
        wave_range(l, h, valid, (flags & ANG_HORIZ) ? G.cols : G.rows, lo, hi);
    }

    // Sums of the rays over part `part` of np of the steps; SEQ: over all np, one
    // part after another.
    template <bool SEQ>
    __device__ __forceinline__ void sum(const GeomDev& G, const T* __restrict__ xp, const T* __restrict__ xTp,
                                        int part, int np, double (&acc)[2]) const {
        auto parts = [&](auto walk) {   // walk(l, h, v): u-weighted sums over [l, h) (see chord_u)
            if constexpr (SEQ) {
                acc[0] = acc[1] = -0.0;   // (-0 + v is v)
#pragma unroll 1
                for (int p = 0; p < np; ++p) {
                    int l = lo, h = hi;
                    part_range(l, h, p, np);
                    double v[2] = {0.0, 0.0};
                    if (l < h) walk(l, h, v);
                    acc[0] += v[0] * A.wmax;
                    acc[1] += v[1] * A.wmax;
                }
            } else {
                int l = lo, h = hi;
                part_range(l, h, part, np);
                acc[0] = acc[1] = 0.0;
                if (l < h) walk(l, h, acc);
                acc[0] *= A.wmax;
                acc[1] *= A.wmax;
            }
        };
        const bool horiz = flags & ANG_HORIZ;
        if (flags & ANG_AXIS) {
            if (horiz) parts([&](int l, int h, double (&v)[2]) { v[0] = ray_sum_axis<true>(G, A, s0, xTp + PAD, l, h); });
            else parts([&](int l, int h, double (&v)[2]) { v[0] = ray_sum_axis<false>(G, A, s0, xp + PAD, l, h); });
        } else if constexpr (PAIR) {
            auto pair = [&](auto hz, const T* img) {
                constexpr bool H = decltype(hz)::value;
                const bool sw = pair_swap<H>(A);
                parts([&](int l, int h, double (&v)[2]) {
                    double w[2];
                    ray_pair<H>(G, A, sw ? s1 : s0, img, l, h, w);
                    // The upper ray multiplies one pixel more per band than it
                    // would by itself, by weight 0: NaN where that is not
                    // finite, so it is then summed again by itself.  (A finite
                    // sum has met finite pixels alone.)
                    const bool finite = fabs(w[1]) < __builtin_inf();
                    if (__any(!finite)) {
                        const double own = ray_split<H>(G, A, sw ? s0 : s1, img, l, h);
                        if (!finite) w[1] = own;
                    }
                    v[0] = sw ? w[1] : w[0];
                    v[1] = sw ? w[0] : w[1];
                });
            };
            if (horiz) pair(std::true_type{}, xTp + PAD);
            else pair(std::false_type{}, xp + PAD);
        } else {
            if (horiz) parts([&](int l, int h, double (&v)[2]) { v[0] = ray_split<true>(G, A, s0, xTp + PAD, l, h); });
            else parts([&](int l, int h, double (&v)[2]) { v[0] = ray_split<false>(G, A, s0, xp + PAD, l, h); });
        }
    }

    // Stores the rays whose whole sums are acc (partials index pidx).
    __device__ __forceinline__ void store(const GeomDev& G, const double (&acc)[2], const RayOut& o, int pidx) const {
        double r2 = project_value(G, A.row, A.wmax, k, valid, acc[0], o);
        if (PAIR) r2 += project_value(G, A.row, A.wmax, k + 1, valid2, acc[1], o);
        project_partial(r2, o, pidx);
    }
};

// Parts, waves and ray workgroups of the form that copies of type T take.
template <class T>
__host__ __device__ inline int ray_parts(const GeomDev& G) { return sizeof(T) == 4 ? G.fparts : G.parts; }
template <class T>
inline bool ray_mem(const GeomDev& G) { return sizeof(T) == 4 ? G.fparts > WG_PARTS : G.pmem != 0; }
template <class T>
__host__ __device__ inline int ray_waves(const GeomDev& G) { return sizeof(T) == 4 ? G.fwaves : G.nwaves; }
template <class T>
inline int ray_wgs(const GeomDev& G) { return sizeof(T) == 4 ? G.fwg : G.nwg; }

// Rays of ray workgroup wg (entries 4 wg .. 4 wg + 3 of the wave table), whole.
// Parts that do not go through memory: a workgroup has four waves per part: waves
// 4 p .. sum part p, and the parts are added in order through LDS (no pass over
// memory, no second launch).  The batched form (SEQ) has one wave per table
// entry, which sums the parts one after another: the same sums.
template <bool SEQ, class T>
__device__ __forceinline__ void project_body(const GeomDev& G, const AngleDev* __restrict__ ang,
                                             const WaveDev* __restrict__ waves,
                                             const T* __restrict__ xp,
                                             const T* __restrict__ xTp,
                                             const RayOut& o, int wg) {
    constexpr int NR = LaneRays<T>::PAIR ? 2 : 1;
    __shared__ double parts[WG_PARTS - 1][NR][256];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int np = ray_parts<T>(G);
    LaneRays<T> R;
    R.set(G, ang, waves, 4 * wg + (w & 3), ray_waves<T>(G));
    double acc[2];
    if constexpr (SEQ) {
        R.template sum<true>(G, xp, xTp, 0, np, acc);
    } else {
        R.template sum<false>(G, xp, xTp, w >> 2, np, acc);
        if (np > 1) {
            const int t = threadIdx.x & 255;
            if (w >= 4) {
#pragma unroll
                for (int r = 0; r < NR; ++r) parts[(w >> 2) - 1][r][t] = acc[r];
            }
            __syncthreads();
            if (w >= 4) return;
            for (int p = 1; p < np; ++p) {
#pragma unroll
                for (int r = 0; r < NR; ++r) acc[r] += parts[p - 1][r][t];
            }
        }
    }
    R.store(G, acc, o, wg);
}

// Part `part` of the rays of workgroup wg (parts through memory), to
// seg[(part*nA + ai)*nB + k] (ai: class-sorted table index); the combine step
// adds the parts in order.  The parts of a large image run one after another
// (part the slowest grid index), so the resident waves read a band of it.
template <class T>
__device__ __forceinline__ void project_part_body(const GeomDev& G, const AngleDev* __restrict__ ang,
                                                  const WaveDev* __restrict__ waves,
                                                  const T* __restrict__ xp,
                                                  const T* __restrict__ xTp,
                                                  double* __restrict__ seg, int wg, int part) {
    LaneRays<T> R;
    R.set(G, ang, waves, 4 * wg + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), ray_waves<T>(G));
    double acc[2];
    R.template sum<false>(G, xp, xTp, part, ray_parts<T>(G), acc);
    double* v = seg + ((size_t)part * G.nA + R.ai) * G.nB + R.k;
    if (R.valid) v[0] = acc[0];
    if (R.PAIR && R.valid2) v[1] = acc[1];
}

// Sum of the parts of the rays of combine block (bx, by): angle bx of the
// class-sorted table, 256-bin chunk by; then the store (partials index
// by * gx + bx).
__device__ __forceinline__ void project_comb_body(const GeomDev& G, const AngleDev* __restrict__ ang,
                                                  const double* __restrict__ seg, const RayOut& o,
                                                  int parts, int bx, int by, int gx) {
    const double wmax = ang[bx].wmax;
    const int k = by * 256 + threadIdx.x;
    const bool valid = k < G.nB;
    double acc = 0.0;
    if (valid) {
        const double* v = seg + (size_t)bx * G.nB + k;
        const size_t stride = (size_t)G.nA * G.nB;
        for (int j = 0; j < parts; ++j) acc += v[j * stride];
    }
    project_partial(project_value(G, ang[bx].row, wmax, k, valid, acc, o), o, by * gx + bx);
}

// The same sums of at most WG_PARTS parts (one ray per lane) for ray workgroup wg,
// with the partials of project_body.
__device__ __forceinline__ void project_sum_body(const GeomDev& G, const AngleDev* __restrict__ ang,
                                                 const WaveDev* __restrict__ waves,
                                                 const double* __restrict__ seg, const RayOut& o, int wg) {
    const int wi = 4 * wg + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const WaveDev W = waves[wi < G.nwaves ? wi : 0];
    int ai, k;
    const bool valid = wave_ray(W, threadIdx.x & 63, G.nB, ai, k) && wi < G.nwaves;
    if (!valid) ai = W.a0, k = 0;
    const double* v = seg + (size_t)ai * G.nB + k;
    const size_t stride = (size_t)G.nA * G.nB;
    double acc = valid ? v[0] : 0.0;
    for (int j = 1; valid && j < G.parts; ++j) acc += v[j * stride];
    project_partial(project_value(G, ang[ai].row, ang[ai].wmax, k, valid, acc, o), o, wg);
}

// 256 threads per part (at most WG_PARTS), one workgroup per ray workgroup.
template <class T>
__global__ __launch_bounds__(256 * WG_PARTS, sizeof(T) == 4 ? 4 : 8) void k_project(GeomDev G, const AngleDev* __restrict__ ang,
                                                              const WaveDev* __restrict__ waves,
                                                              const T* __restrict__ xp,
                                                              const T* __restrict__ xTp,
                                                              RayOut o, const int* __restrict__ ord,
                                                              const int* __restrict__ halt) {
    if (halt && *halt) return;
    project_body<false, T>(G, ang, waves, xp, xTp, o, ord[blockIdx.x]);
}

// grid (ray workgroups, parts): blockIdx.y is the part, so the parts run in order.
template <class T>
__global__ __launch_bounds__(256, sizeof(T) == 4 ? 4 : 8) void k_project_part(GeomDev G, const AngleDev* __restrict__ ang,
                                                      const WaveDev* __restrict__ waves,
                                                      const T* __restrict__ xp,
                                                      const T* __restrict__ xTp,
                                                      double* __restrict__ seg,
                                                      const int* __restrict__ ord,
                                                      const int* __restrict__ halt) {
    if (halt && *halt) return;
    project_part_body<T>(G, ang, waves, xp, xTp, seg, ord[blockIdx.x], blockIdx.y);
}

__global__ __launch_bounds__(256) void k_project_comb(GeomDev G, const AngleDev* __restrict__ ang,
                                                      const double* __restrict__ seg, RayOut o, int parts,
                                                      const int* __restrict__ halt) {
    if (halt && *halt) return;
    project_comb_body(G, ang, seg, o, parts, blockIdx.x, blockIdx.y, gridDim.x);
}

__global__ __launch_bounds__(256) void k_project_sum(GeomDev G, const AngleDev* __restrict__ ang,
                                                     const WaveDev* __restrict__ waves,
                                                     const double* __restrict__ seg, RayOut o,
                                                     const int* __restrict__ halt) {
    if (halt && *halt) return;
    project_sum_body(G, ang, waves, seg, o, blockIdx.x);
}

// residual: rpd = R xh - b (float64) with f partials; else w = R z (float64)
// with the partials of w^T q, both into pf.
__device__ __forceinline__ RayOut batch_out(const SliceDev& S, bool residual) {
    RayOut o;
    o.partials = gmem(S.pf);
    if (residual) {
        o.b = gmem(S.b);
        o.outpd = gmem(S.rpd);
    } else {
        o.dq = gmem(S.q);
        o.wout = gmem(S.w);
    }
    return o;
}

// The slices without pmem: item lin runs ray workgroup lin of the
// order, whole, a wave summing its rays' parts one after another.  Apart from the split slices' body, and with the loop over the
// parts inside each walk, it fits eight waves per SIMD (one kernel for both,
// six: 16 slices of 128^2 to 512^2 246 -> 217 us; part sums through memory and
// a second launch 223 + 22).
__global__ __launch_bounds__(256, 8) void kb_project(const SliceDev* __restrict__ sl, ItemTable t,
                                                  int residual) {
    for_items(t, [&](int s, int lin) {
        const SliceDev& S = sl[s];
        if (gmem(S.sc)->halt) return;
        const GeomDev G = S.G;
        project_body<true, double>(G, cmem(S.ang), cmem(S.pwave), gmem(S.xp), gmem(S.xTp), batch_out(S, residual),
                                   cmem(S.pord)[lin]);
    });
}

// The same with the parts side by side in the workgroup, as the single-slice
// launch: one item per workgroup, since the waves of the parts beyond the first
// end before its sums are stored (and those of parts that the slice does not
// have at once).
__global__ __launch_bounds__(256 * WG_PARTS, 8) void kb_project_wg(const SliceDev* __restrict__ sl, ItemTable t,
                                                              int residual) {
    const uint32_t it = t.items[blockIdx.x];
    if (it == ITEM_NONE) return;
    const SliceDev& S = sl[it >> ITEM_SHIFT];
    if (gmem(S.sc)->halt) return;
    const GeomDev G = S.G;
    if ((int)(threadIdx.x >> 8) >= G.parts) return;
    project_body<false, double>(G, cmem(S.ang), cmem(S.pwave), gmem(S.xp), gmem(S.xTp), batch_out(S, residual),
                                cmem(S.pord)[it & ITEM_MASK]);
}

// The slices with pmem: item lin = part * (ray workgroups) + i runs that part of ray
// workgroup i of the order.
__global__ __launch_bounds__(256, 8) void kb_project_part(const SliceDev* __restrict__ sl, ItemTable t) {
    for_items(t, [&](int s, int lin) {
        const SliceDev& S = sl[s];
        if (gmem(S.sc)->halt) return;
        const GeomDev G = S.G;
        project_part_body<double>(G, cmem(S.ang), cmem(S.pwave), gmem(S.xp), gmem(S.xTp), gmem(S.seg),
                                  cmem(S.pord)[lin % G.nwg], lin / G.nwg);
    });
}

// The combine step of the slices with more than WG_PARTS parts; virtual block
// by * nA + bx.
__global__ __launch_bounds__(256) void kb_project_comb(const SliceDev* __restrict__ sl, ItemTable t,
                                                       int residual) {
    for_items(t, [&](int s, int lin) {
        const SliceDev& S = sl[s];
        if (gmem(S.sc)->halt) return;
        const GeomDev G = S.G;
        const int gx = G.nA;
        project_comb_body(G, cmem(S.ang), gmem(S.seg), batch_out(S, residual), G.parts, lin % gx, lin / gx, gx);
    });
}

// That of the slices with pmem and fewer; virtual block: the ray workgroup.
__global__ __launch_bounds__(256) void kb_project_sum(const SliceDev* __restrict__ sl, ItemTable t, int residual) {
    for_items(t, [&](int s, int lin) {
        const SliceDev& S = sl[s];
        if (gmem(S.sc)->halt) return;
        const GeomDev G = S.G;
        project_sum_body(G, cmem(S.ang), cmem(S.pwave), gmem(S.seg), batch_out(S, residual), lin);
    });
}

void launch_project_b(hipStream_t st, const SliceDev* sl, const ProjectTables& T, bool residual) {
    const int r = residual ? 1 : 0;
    if (T.t.n > 0 && T.wg_parts > 0)
        hipLaunchKernelGGL(kb_project_wg, dim3(T.t.n), dim3(256 * T.wg_parts), 0, st, sl, T.t, r);
    else if (T.t.n > 0)
        hipLaunchKernelGGL(kb_project, dim3(T.t.grid), dim3(256), 0, st, sl, T.t, r);
    if (T.tp.n > 0) hipLaunchKernelGGL(kb_project_part, dim3(T.tp.grid), dim3(256), 0, st, sl, T.tp);
    if (T.tc.n > 0) hipLaunchKernelGGL(kb_project_comb, dim3(T.tc.grid), dim3(256), 0, st, sl, T.tc, r);
    if (T.ts.n > 0) hipLaunchKernelGGL(kb_project_sum, dim3(T.ts.grid), dim3(256), 0, st, sl, T.ts, r);
}

template <class T>
void launch_project_form(hipStream_t st, const GeomDev& G, const AngleDev* ang, const WaveDev* waves,
                         const T* xp, const T* xTp, const RayOut& o, double* seg, const int* ord,
                         const int* halt) {
    const int parts = ray_parts<T>(G);
    if (ray_mem<T>(G)) {
        hipLaunchKernelGGL((k_project_part<T>), dim3(ray_wgs<T>(G), parts), dim3(256), 0, st, G, ang, waves, xp,
                           xTp, seg, ord, halt);
        if (parts > WG_PARTS)
            hipLaunchKernelGGL(k_project_comb, dim3(G.nA, (G.nB + 255) / 256), dim3(256), 0, st, G,
                               ang, (const double*)seg, o, parts, halt);
        else
            hipLaunchKernelGGL(k_project_sum, dim3(G.nwg), dim3(256), 0, st, G, ang, waves, (const double*)seg, o, halt);
        return;
    }
    hipLaunchKernelGGL((k_project<T>), dim3(ray_wgs<T>(G)), dim3(256 * parts), 0, st, G, ang, waves, xp, xTp, o, ord,
                       halt);
}

void launch_project(hipStream_t st, const GeomDev& G, const AngleDev* ang, const WaveDev* waves,
                    const double* xp, const double* xTp, const RayOut& o, double* seg, const int* ord,
                    const int* halt) {
    launch_project_form<double>(st, G, ang, waves, xp, xTp, o, seg, ord, halt);
}

void launch_project32(hipStream_t st, const GeomDev& G, const AngleDev* ang, const WaveDev* waves,
                      const float* zp, const float* zTp, const RayOut& o, double* seg, const int* ord,
                      const int* halt) {
    launch_project_form<float>(st, G, ang, waves, zp, zTp, o, seg, ord, halt);
}

// Padded copy of a caller's sinogram for R^T, each row times its angle's wmax
// (the scaling bp_class expects), pads written as zeros; one workgroup per
// entry of the angle table.
__global__ __launch_bounds__(256) void k_pad_sino(GeomDev G, const AngleDev* __restrict__ ang,
                                                  const float* __restrict__ y,
                                                  float* __restrict__ yp) {
    const int a = ang[blockIdx.x].row;
    const double wmax = ang[blockIdx.x].wmax;
    float* row = yp + (size_t)a * G.pitchB;
    for (int k = threadIdx.x; k < G.pitchB; k += 256) {
        const int kk = k - PAD;
        row[k] = kk >= 0 && kk < G.nB ? (float)((double)y[(size_t)a * G.nB + kk] * wmax) : 0.0f;
    }
}

void launch_pad_sino(hipStream_t st, const GeomDev& G, const AngleDev* ang, const float* y,
                     float* yp) {
    hipLaunchKernelGGL(k_pad_sino, dim3(G.nA), dim3(256), 0, st, G, ang, y, yp);
}

// ---- backward gather ----------------------------------------------------------
// Sum over the angles [beg, end) of one class for pixel row yi and the PX
// pixels xj[u] of this lane.  The angle and its sinogram row are wave-uniform
// (scalar loads); lanes differ only in the pixel.  The padded sinogram rows
// arrive multiplied by their angle's wmax (project_value, k_pad_sino), so each
// candidate adds u * y' with the u of chord_u: the same weights as the
// projector's wmax * u.
//
// Candidate window: the NB bins from padded index trunc(kf), kf = t / ds + kb
// with t = xj c + yi s (A.kb carries the - s0 / ds, the half-width hb of the
// nonzero band plus a margin, and the + 1 + PAD of the padded index; see
// bp_kf).  For oblique angles kf = fma(xj, c / ds, yi s / ds + kb), the
// second term shared by the lane's pixels, and the first candidate's offset
// s_k - t is dc - ds fract(kf) with dc = ds (1 - hb) (the same value as
// s_k - t up to the rounding of kf, ~1e-13 pixel); the next ones follow by
// + ds.  For axis-parallel angles the offset must be
// exact -- a ray on a pixel edge takes half the pixel -- so s_k is formed from
// the bin index as in bin_pos and t is exact.  A window index below the row
// or past it reads 0 (pads and out-of-row reads), so such candidates add 0.
template <bool AXIS, int NB, class TY, int PX>
__device__ __forceinline__ void bp_class(const GeomDev& G, const AngleDev* __restrict__ ang,
                                         int beg, int end, const TY* __restrict__ yp,
                                         const double* xj, double yi, double* acc) {
    const int rowbytes = G.pitchB * (int)sizeof(TY);
    // 1/ds held in a vector register, so the index FMA's one scalar operand
    // can be the angle's kb (an FMA reads at most one scalar register)
    double ids = G.inv_ds;
    asm volatile("" : "+v"(ids));
    double ds = G.ds;   // likewise for the offset FMA, whose addend is the angle's dc
    asm volatile("" : "+v"(ds));
#pragma unroll 2
    for (int a = beg; a < end; ++a) {
        const AngleDev A = ang[a];
        const __amdgpu_buffer_rsrc_t rs = row_rsrc(yp + (size_t)A.row * G.pitchB, rowbytes);
        const double ys = AXIS ? yi * A.s : 0.0;
        const double kc = AXIS ? 0.0 : bp_kc(yi, A);
        TY v[PX][NB];
        double d0[PX], tt[PX];
        int oo[PX];
#pragma unroll
        for (int u = 0; u < PX; ++u) {
            double kf;
            if (AXIS) {
                tt[u] = fma(xj[u], A.c, ys);
                kf = bp_kf(tt[u], ids, A.kb);
            } else {
                kf = bp_kf_oblique(xj[u], kc, A);
            }
            const int o = (int)kf;
            row_load<TY, NB>(rs, (unsigned)o, v[u]);
            if (AXIS) oo[u] = o;
            else d0[u] = fma(__builtin_amdgcn_fract(kf), -ds, A.dc);
        }
#pragma unroll
        for (int u = 0; u < PX; ++u) {
            double d = AXIS ? 0.0 : d0[u];
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                if (AXIS) d = bin_pos((double)(oo[u] - PAD + q), G) - tt[u];
                acc[u] = fma(chord_u<AXIS>(d, A.einv, A.inv), (double)v[u][q], acc[u]);
                if (!AXIS) d += ds;
            }
        }
    }
}

// Share w of n of the range [beg, end).
__device__ __forceinline__ void split_range(int beg, int end, int w, int n, int& b, int& e) {
    const int len = end - beg;
    b = beg + (len * w) / n;
    e = beg + (len * (w + 1)) / n;
}

// Where R^T's image goes: float32 (f), or float64 (d), there rounded to a
// float32 value with round.
struct BpOut {
    float* f;
    double* d;
    bool round;
    __device__ __forceinline__ void put(size_t p, double v) const {
        if (d) d[p] = round ? (double)(float)v : v;
        else f[p] = (float)v;
    }
};

// out[i][j] = (R^T y)_{ij} from the padded sinogram yp.  A workgroup owns an
// 8 x 8PX pixel tile (PX pixels, 8 columns apart, per lane); its wave w sums
// the w-th quarter of every angle class, and the four partial sums are added
// in wave order through LDS.
template <int NB, class TY, int PX>
__device__ __forceinline__ void backproject_body(const GeomDev& G, const AngleDev* __restrict__ ang,
                                                 const TY* __restrict__ yp, BpOut out, int bx, int by) {
    __shared__ double part[BP_SPLIT][PX][64];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i = by * BP_TILE + (lane >> 3);
    const int j0 = bx * 8 * PX + (lane & 7);
    const double yi = G.yoff - (double)i;
    double acc[PX], xj[PX];
#pragma unroll
    for (int u = 0; u < PX; ++u) {
        acc[u] = 0.0;
        xj[u] = (double)(j0 + 8 * u) - G.xoff;
    }
    int b, e;
    split_range(G.cls[0], G.cls[2], w, BP_SPLIT, b, e);   // oblique angles of both orientations
    bp_class<false, NB, TY, PX>(G, ang, b, e, yp, xj, yi, acc);
    split_range(G.cls[2], G.cls[4], w, BP_SPLIT, b, e);   // axis-parallel angles
    bp_class<true, NB, TY, PX>(G, ang, b, e, yp, xj, yi, acc);
#pragma unroll
    for (int u = 0; u < PX; ++u) part[w][u][lane] = acc[u];
    __syncthreads();
    if (w == 0) {
#pragma unroll
        for (int u = 0; u < PX; ++u) {
            const int j = j0 + 8 * u;
            const double tot =
                ((part[0][u][lane] + part[1][u][lane]) + part[2][u][lane]) + part[3][u][lane];
            if (i < G.rows && j < G.cols) out.put((size_t)i * G.cols + j, tot * G.pixel);
        }
    }
}

// ---- 2 x 2 pixel blocks --------------------------------------------------------
// The oblique angles [beg, end) for the lane's NQ blocks of 2 x 2 pixels with
// centres (xc[n], yc).  Bound: the float64 VALU (about 9 instructions per pixel
// and angle).  A pixel at a time costs a window index and a gather each, and
// the vector L1's access rate (16 or more accesses per gather whatever its
// width) held R^T at 11 instructions and one gather per pixel.  At about unit
// bin spacing a block's four footprints lie within three bins (bp_quad_table
// checks it), so one index and one 12-byte gather (24 bytes in two from a
// float64 sinogram) serve four pixels; only 10 of the 12 pixel-bin pairs can
// meet, and half of those lie on a known side of the pixel's centre, where
// the weight is one add with output clamp.  512^2 x 720 x 725, float64
// residual: 0.106 -> 0.059 ms (189M pixel-angles, 3.2e12 per second); float32
// sinogram with its padding pass 0.097 -> 0.070; 2048^2 x 2864: 5.3 -> 3.3 ms.
// The accumulators are kept in the order A, B, C, D of BpAngle, which only
// changes between runs of angles (the signs of cos and sin, and which is
// larger); acc holds each block's pixels 2 r + c (row r, column c).  One angle
// per iteration with two blocks, or many waves of one, hides the scalar loads
// of its constants; two angles per iteration ran out of scalar registers.
template <class TY>
struct QuadBins;
template <>
struct QuadBins<float> {
    static __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, int o, double (&v)[3]) {
        typedef float f3v __attribute__((ext_vector_type(3)));
        const f3v t = __builtin_bit_cast(f3v, __builtin_amdgcn_raw_buffer_load_b96(r, 4u * (unsigned)o, 0, 0));
        v[0] = (double)t.x;
        v[1] = (double)t.y;
        v[2] = (double)t.z;
    }
};
template <>
struct QuadBins<double> {
    static __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, int o, double (&v)[3]) {
        const unsigned off = 8u * (unsigned)o;
        const d2v t = __builtin_bit_cast(d2v, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
        v[0] = t.x;
        v[1] = t.y;
        v[2] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off + 16u, 0, 0));
    }
};

__device__ __forceinline__ void swap_acc(double& a, double& b) {
    const double t = a;
    a = b;
    b = t;
}

template <class TY, int NQ>
__device__ __forceinline__ void bp_quads(const GeomDev& G, const BpAngle* __restrict__ quad, int beg, int end,
                                         const TY* __restrict__ yp, const double (&xc)[NQ], double yc,
                                         double (&acc)[NQ][4]) {
    const int rowbytes = G.pitchB * (int)sizeof(TY);
    for (int a = beg; a < end;) {
        const int run = quad[a].run;
        const int stop = min(end, run >> BP_CODE_BITS);
        // to the corners' order (bp_quad_corner), and back after the run
        const bool fx = run & BP_FLIP_X, fy = run & BP_FLIP_Y, vert = run & BP_VERT;
#pragma unroll
        for (int n = 0; n < NQ; ++n) {
            double (&v)[4] = acc[n];
            if (fx) swap_acc(v[0], v[1]), swap_acc(v[2], v[3]);
            if (fy) swap_acc(v[0], v[2]), swap_acc(v[1], v[3]);
            if (vert) swap_acc(v[1], v[2]);
        }
#pragma unroll 1
        for (int q = a; q < stop; ++q) {
            const BpAngle Q = quad[q];
            const __amdgpu_buffer_rsrc_t rs = row_rsrc(yp + (size_t)Q.row * G.pitchB, rowbytes);
            double v[NQ][3], w[NQ];
#pragma unroll
            for (int n = 0; n < NQ; ++n) {
                const double kf = bp_quad_kf(xc[n], yc, Q);
                QuadBins<TY>::load(rs, (int)kf, v[n]);
                w[n] = bp_quad_w(__builtin_amdgcn_fract(kf), Q);
            }
#pragma unroll
            for (int n = 0; n < NQ; ++n) {
                double u2[2], u3[3];
                double &aA = acc[n][0], &aB = acc[n][1], &aC = acc[n][2], &aD = acc[n][3];
                bp_quad_a(Q, w[n], u2);
                aA = fma(u2[0], v[n][0], aA);
                aA = fma(u2[1], v[n][1], aA);
                bp_quad_d(Q, w[n], u2);
                aD = fma(u2[0], v[n][1], aD);
                aD = fma(u2[1], v[n][2], aD);
                bp_quad_b(Q, w[n], u3);
                aB = fma(u3[0], v[n][0], aB);
                aB = fma(u3[1], v[n][1], aB);
                aB = fma(u3[2], v[n][2], aB);
                bp_quad_c(Q, w[n], u3);
                aC = fma(u3[0], v[n][0], aC);
                aC = fma(u3[1], v[n][1], aC);
                aC = fma(u3[2], v[n][2], aC);
            }
        }
#pragma unroll
        for (int n = 0; n < NQ; ++n) {
            double (&v)[4] = acc[n];
            if (vert) swap_acc(v[1], v[2]);
            if (fy) swap_acc(v[0], v[2]), swap_acc(v[1], v[3]);
            if (fx) swap_acc(v[0], v[1]), swap_acc(v[2], v[3]);
        }
        a = stop;
    }
}

// R^T over 2 x 2 blocks: a workgroup owns NQ 16 x 16 pixel tiles side by side
// (tile `id` in the order of bp_tile_of), lane l block (l / 8, l % 8) of each.
// The angles are split into G.bp_shares shares; wave w of the workgroup's NW
// sums shares w, w + NW, ..., and the shares are added in order through LDS, so
// the result does not depend on NW or NQ.
template <class TY, int NW, int NQ>
__device__ __forceinline__ void bp_quad_body(const GeomDev& G, const AngleDev* __restrict__ ang,
                                             const BpAngle* __restrict__ quad, const TY* __restrict__ yp,
                                             BpOut out, int id) {
    constexpr int PX = 4;
    extern __shared__ double part[];   // [shares][NQ][PX][64]
    const int gx = (G.cols + NQ * BPQ_TILE - 1) / (NQ * BPQ_TILE), gy = (G.rows + BPQ_TILE - 1) / BPQ_TILE;
    int bx, by;
    bp_tile_of(id, gx, gy, bx, by);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i0 = by * BPQ_TILE + 2 * (lane >> 3), j0 = bx * NQ * BPQ_TILE + 2 * (lane & 7);
    const double yc = G.yoff - ((double)i0 + 0.5);
    double xc[NQ];
#pragma unroll
    for (int n = 0; n < NQ; ++n) xc[n] = (double)(j0 + n * BPQ_TILE) + 0.5 - G.xoff;
    const int shares = G.bp_shares;
    for (int sh = wave; sh < shares; sh += NW) {
        double acc[NQ][PX];
#pragma unroll
        for (int n = 0; n < NQ; ++n)
#pragma unroll
            for (int u = 0; u < PX; ++u) acc[n][u] = 0.0;
        int b, e;
        split_range(G.cls[0], G.cls[2], sh, shares, b, e);   // oblique angles of both orientations
        bp_quads<TY, NQ>(G, quad, b, e, yp, xc, yc, acc);
        split_range(G.cls[2], G.cls[4], sh, shares, b, e);   // axis-parallel angles
        if (b < e) {
#pragma unroll
            for (int n = 0; n < NQ; ++n)
#pragma unroll
                for (int p = 0; p < PX; ++p) {
                    const double xj[1] = {xc[n] + ((p & 1) ? 0.5 : -0.5)};
                    bp_class<true, 2, TY, 1>(G, ang, b, e, yp, xj, yc + ((p & 2) ? -0.5 : 0.5), &acc[n][p]);
                }
        }
#pragma unroll
        for (int n = 0; n < NQ; ++n)
#pragma unroll
            for (int u = 0; u < PX; ++u) part[((sh * NQ + n) * PX + u) * 64 + lane] = acc[n][u];
    }
    __syncthreads();
    for (int m = wave; m < NQ * PX; m += NW) {
        const int n = m / PX, p = m % PX;
        double tot = part[m * 64 + lane];
        for (int sh = 1; sh < shares; ++sh) tot += part[(sh * NQ * PX + m) * 64 + lane];
        const int i = i0 + (p >> 1), j = j0 + n * BPQ_TILE + (p & 1);
        const bool in = i < G.rows && j < G.cols, finite = fabs(tot) < __builtin_inf();
        if (__any(in && !finite)) {
            // A block multiplies bins that only its other pixels meet by weight 0,
            // which is NaN for a bin that is not finite: such a pixel is summed
            // again over its own bins.  (A finite sum has met finite bins alone.)
            const double xj[1] = {xc[n] + ((p & 1) ? 0.5 : -0.5)}, yi = yc + ((p & 2) ? -0.5 : 0.5);
            double own = 0.0;
            bp_class<false, 2, TY, 1>(G, ang, G.cls[0], G.cls[2], yp, xj, yi, &own);
            bp_class<true, 2, TY, 1>(G, ang, G.cls[2], G.cls[4], yp, xj, yi, &own);
            if (!finite) tot = own;
        }
        if (in) out.put((size_t)i * G.cols + j, tot * G.pixel);
    }
}

size_t bp_quad_lds(int shares, int nq) { return (size_t)shares * nq * 4 * 64 * sizeof(double); }

__device__ __forceinline__ void run_ride(const ScalarRide& ride) {
    if (ride.ps) scalar_body(OP_SNORM, ride.sc, ride.tr, ride.ps, ride.ns, nullptr, 0);
    if (ride.pf) scalar_body(OP_F, ride.sc, ride.tr, ride.pf, ride.nf, nullptr, 0);
}

template <int NB, class TY, int PX>
__global__ __launch_bounds__(256) void k_backproject(GeomDev G, const AngleDev* __restrict__ ang,
                                                     const TY* __restrict__ yp, BpOut out,
                                                     ScalarRide ride,
                                                     const int* __restrict__ halt) {
    if (halt && *halt) return;
    int bx, by;
    bp_tile_of(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x, gridDim.y, bx, by);
    backproject_body<NB, TY, PX>(G, ang, yp, out, bx, by);
    if (ride.sc && blockIdx.x == 0 && blockIdx.y == 0) run_ride(ride);
}

template <class TY, int NW, int NQ>
__global__ __launch_bounds__(64 * NW) void k_backproject_quad(GeomDev G, const AngleDev* __restrict__ ang,
                                                              const BpAngle* __restrict__ quad,
                                                              const TY* __restrict__ yp, BpOut out,
                                                              ScalarRide ride,
                                                              const int* __restrict__ halt) {
    if (halt && *halt) return;
    bp_quad_body<TY, NW, NQ>(G, ang, quad, yp, out, blockIdx.x);
    if (ride.sc && blockIdx.x == 0) {
        if (threadIdx.x >= 256) return;   // the scalar steps are those of a 256-thread workgroup
        run_ride(ride);
    }
}

// g = R^T rpd from the float64 residual.  NB is the largest candidate count of
// the batch (extra candidates weigh exactly 0).
template <int NB, int PX>
__global__ __launch_bounds__(256) void kb_backproject(const SliceDev* __restrict__ sl, ItemTable t, int round) {
    for_items(t, [&](int s, int lin) {
        const SliceDev& S = sl[s];
        if (gmem(S.sc)->halt) return;
        const GeomDev G = S.G;
        int bx, by;
        bp_tile_of(lin, (G.cols + 8 * PX - 1) / (8 * PX), (G.rows + BP_TILE - 1) / BP_TILE, bx, by);
        backproject_body<NB, double, PX>(G, cmem(S.ang), gmem(S.rpd),
                                         BpOut{nullptr, gmem(S.g), round != 0}, bx, by);
    });
}

// NW waves per workgroup, each summing every NW-th share.
template <int NW, int NQ>
__global__ __launch_bounds__(64 * NW) void kb_backproject_quad(const SliceDev* __restrict__ sl, ItemTable t,
                                                           int round) {
    for_items(t, [&](int s, int lin) {
        const SliceDev& S = sl[s];
        if (gmem(S.sc)->halt) return;
        const GeomDev G = S.G;
        bp_quad_body<double, NW, NQ>(G, cmem(S.ang), cmem(S.quad), gmem(S.rpd),
                                     BpOut{nullptr, gmem(S.g), round != 0}, lin);
    });
}

template <int PX>
void launch_bp_b_px(hipStream_t st, const SliceDev* sl, ItemTable t, int nbmax, int round) {
    switch (nbmax) {
    case 1: hipLaunchKernelGGL((kb_backproject<1, PX>), dim3(t.grid), dim3(256), 0, st, sl, t, round); break;
    case 2: hipLaunchKernelGGL((kb_backproject<2, PX>), dim3(t.grid), dim3(256), 0, st, sl, t, round); break;
    case 3: hipLaunchKernelGGL((kb_backproject<3, PX>), dim3(t.grid), dim3(256), 0, st, sl, t, round); break;
    default: hipLaunchKernelGGL((kb_backproject<4, PX>), dim3(t.grid), dim3(256), 0, st, sl, t, round); break;
    }
}

template <int NW, int NQ>
void launch_bp_b_quad(hipStream_t st, const SliceDev* sl, ItemTable t, int shares, int round) {
    if (t.n > 0)
        hipLaunchKernelGGL((kb_backproject_quad<NW, NQ>), dim3(t.grid), dim3(64 * NW), bp_quad_lds(shares, NQ), st, sl, t,
                           round);
}

void launch_backproject_b(hipStream_t st, const SliceDev* sl, const BackprojectTables& T, bool round) {
    const int rd = round ? 1 : 0;
    // (The wave slots hold the 16 shares of q16_wide tiles at once; more take their
    // shares in two turns, so that workgroups of one CU overlap.  Iteration, 8 / 16
    // waves: 1 x 64^2 85 / 83 us, 4 x 128^2 114 / 109, 1 x 250^2 131 / 124, 2 x 250^2
    // 180 / 184, 16 x 180^2 361 / 396.)
    if (T.q16.n <= T.q16_wide) launch_bp_b_quad<16, 1>(st, sl, T.q16, 16, rd);
    else launch_bp_b_quad<8, 1>(st, sl, T.q16, 16, rd);
    launch_bp_b_quad<8, 1>(st, sl, T.q8, 8, rd);
    launch_bp_b_quad<4, 2>(st, sl, T.q2, 4, rd);
    if (T.pixel.n == 0) return;
    if (T.px == 4) launch_bp_b_px<4>(st, sl, T.pixel, T.nbmax, rd);
    else launch_bp_b_px<2>(st, sl, T.pixel, T.nbmax, rd);
}

template <class TY, int PX>
void launch_bp_px(hipStream_t st, const GeomDev& G, const AngleDev* ang, const TY* yp, BpOut out,
                  const int* halt, const ScalarRide& ride) {
    dim3 grid((G.cols + 8 * PX - 1) / (8 * PX), (G.rows + BP_TILE - 1) / BP_TILE);
    switch (G.nbmax) {
    case 1: hipLaunchKernelGGL((k_backproject<1, TY, PX>), grid, dim3(256), 0, st, G, ang, yp, out, ride, halt); break;
    case 2: hipLaunchKernelGGL((k_backproject<2, TY, PX>), grid, dim3(256), 0, st, G, ang, yp, out, ride, halt); break;
    case 3: hipLaunchKernelGGL((k_backproject<3, TY, PX>), grid, dim3(256), 0, st, G, ang, yp, out, ride, halt); break;
    default: hipLaunchKernelGGL((k_backproject<4, TY, PX>), grid, dim3(256), 0, st, G, ang, yp, out, ride, halt); break;
    }
}

template <class TY, int NW, int NQ>
void launch_bp_quad(hipStream_t st, const GeomDev& G, const AngleDev* ang, const BpAngle* quad, const TY* yp,
                    BpOut out, const int* halt, const ScalarRide& ride) {
    hipLaunchKernelGGL((k_backproject_quad<TY, NW, NQ>), dim3(backproject_tiles(G, G.bp_px)), dim3(64 * NW),
                       bp_quad_lds(G.bp_shares, NQ), st, G, ang, quad, yp, out, ride, halt);
}

// Blocks: one wave per share (two tiles per wave go with 4 shares, see
// backproject_shape).
template <class TY>
void launch_bp(hipStream_t st, const GeomDev& G, const AngleDev* ang, const BpAngle* quad, const TY* yp,
               BpOut out, const int* halt, const ScalarRide& ride) {
    if (G.bp_quad && G.bp_nq == 2) launch_bp_quad<TY, 4, 2>(st, G, ang, quad, yp, out, halt, ride);
    else if (G.bp_quad && G.bp_shares == 8) launch_bp_quad<TY, 8, 1>(st, G, ang, quad, yp, out, halt, ride);
    else if (G.bp_quad) launch_bp_quad<TY, 16, 1>(st, G, ang, quad, yp, out, halt, ride);
    else if (G.bp_px == 4) launch_bp_px<TY, 4>(st, G, ang, yp, out, halt, ride);
    else launch_bp_px<TY, 2>(st, G, ang, yp, out, halt, ride);
}

void launch_backproject(hipStream_t st, const GeomDev& G, const AngleDev* ang, const BpAngle* quad,
                        const float* yp, float* out, const int* halt, const ScalarRide& ride) {
    launch_bp(st, G, ang, quad, yp, BpOut{out, nullptr, false}, halt, ride);
}

void launch_backproject(hipStream_t st, const GeomDev& G, const AngleDev* ang, const BpAngle* quad,
                        const double* yp, float* out, double* outd, bool round, const int* halt,
                        const ScalarRide& ride) {
    launch_bp(st, G, ang, quad, yp, BpOut{out, outd, round}, halt, ride);
}

}  // namespace sp
