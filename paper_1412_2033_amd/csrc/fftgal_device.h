// Device helpers shared by the HIP sources: complex arithmetic, in-register DFTs,
// in-place LDS stages of the compile-time lengths, the admissible basis,
// work-group sums, problem lookup and the dispatch of timed launches.
#pragma once

#include "fftgal_internal.h"

#include <type_traits>

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

namespace fftgal {
namespace {

template <typename T> struct VecOf;
template <> struct VecOf<float> { using type = float2; };
template <> struct VecOf<double> { using type = double2; };

template <typename T> using Vt = typename VecOf<T>::type;

// The argument tables hold generic pointers; operands known to live in device
// global memory are cast to that address space so that the compiler emits
// global (not flat) accesses and may move them past LDS accesses.
template <typename T> __device__ __forceinline__ __attribute__((address_space(1))) T *gbl(T *p) {
    return (__attribute__((address_space(1))) T *)(p);
}

template <typename T>
__device__ __forceinline__ Vt<T> mk(T a, T b) {
    Vt<T> v;
    v.x = a;
    v.y = b;
    return v;
}
// complex loads and stores through global-address-space pointers, as one
// 8- or 16-byte access of a native two-element vector
template <typename V> struct ScalarOf;
template <> struct ScalarOf<float2> { using type = float; };
template <> struct ScalarOf<double2> { using type = double; };
template <typename S> using NVec2 = S __attribute__((ext_vector_type(2)));
template <typename V> __device__ __forceinline__ V gld(const __attribute__((address_space(1))) V *p) {
    using S = typename ScalarOf<V>::type;
    const NVec2<S> w = *reinterpret_cast<const __attribute__((address_space(1))) NVec2<S> *>(p);
    V v;
    v.x = w.x;
    v.y = w.y;
    return v;
}
template <typename V> __device__ __forceinline__ void gst(__attribute__((address_space(1))) V *p, V v) {
    using S = typename ScalarOf<V>::type;
    NVec2<S> w;
    w.x = v.x;
    w.y = v.y;
    *reinterpret_cast<__attribute__((address_space(1))) NVec2<S> *>(p) = w;
}
template <typename V> __device__ __forceinline__ V cadd(V a, V b) {
    a.x += b.x;
    a.y += b.y;
    return a;
}
template <typename V> __device__ __forceinline__ V csub(V a, V b) {
    a.x -= b.x;
    a.y -= b.y;
    return a;
}
template <typename V> __device__ __forceinline__ V cmul(V a, V b) {
    V r;
    r.x = a.x * b.x - a.y * b.y;
    r.y = a.x * b.y + a.y * b.x;
    return r;
}

// cos(2 pi j / R) and sin(2 pi j / R), 0 <= j <= (R - 1) / 2.
template <int R> __device__ constexpr double ccos(int j);
template <int R> __device__ constexpr double csin(int j);
template <> __device__ constexpr double ccos<3>(int j) { return j == 0 ? 1.0 : -0.5; }
template <> __device__ constexpr double csin<3>(int j) {
    return j == 0 ? 0.0 : 0.86602540378443864676372317075294;
}
template <> __device__ constexpr double ccos<5>(int j) {
    return j == 0 ? 1.0 : j == 1 ? 0.30901699437494742410229341718282 : -0.80901699437494742410229341718282;
}
template <> __device__ constexpr double csin<5>(int j) {
    return j == 0 ? 0.0 : j == 1 ? 0.95105651629515357211643933337938 : 0.58778525229247312916870595463907;
}
template <> __device__ constexpr double ccos<7>(int j) {
    return j == 0 ? 1.0
         : j == 1 ? 0.62348980185873353052500488400424
         : j == 2 ? -0.22252093395631440428890256449680
                  : -0.90096886790241912623610231950745;
}
template <> __device__ constexpr double csin<7>(int j) {
    return j == 0 ? 0.0
         : j == 1 ? 0.78183148246802980870844452667406
         : j == 2 ? 0.97492791218182360701813168299393
                  : 0.43388373911755812047576833284836;
}

constexpr double kPiD = 3.14159265358979323846;
constexpr double cx_sin_small(double x) {
    double x2 = x * x, t = x, s = x;
    for (int k = 1; k < 14; ++k) {
        t *= -x2 / ((2.0 * k) * (2.0 * k + 1.0));
        s += t;
    }
    return s;
}
constexpr double cx_cos_small(double x) {
    double x2 = x * x, t = 1.0, s = 1.0;
    for (int k = 1; k < 14; ++k) {
        t *= -x2 / ((2.0 * k - 1.0) * (2.0 * k));
        s += t;
    }
    return s;
}
// cos and sin of 2 pi j / R by exact quadrant reduction of the rational j/R
// and Taylor series on [0, pi/4] (evaluated at compile time).
template <int R> struct TrigTab {
    double c[R], s[R];
    constexpr TrigTab() : c(), s() {
        for (int j = 0; j < R; ++j) {
            const int q = (4 * j) / R, r = 4 * j - q * R;
            double cc = 0.0, ss = 0.0;
            if (2 * r <= R) {
                const double t = (kPiD / 2) * r / R;
                cc = cx_cos_small(t);
                ss = cx_sin_small(t);
            } else {
                const double u = (kPiD / 2) * (R - r) / R;
                cc = cx_sin_small(u);
                ss = cx_cos_small(u);
            }
            c[j] = q == 0 ? cc : q == 1 ? -ss : q == 2 ? -cc : ss;
            s[j] = q == 0 ? ss : q == 1 ? cc : q == 2 ? -ss : -cc;
        }
    }
};
template <int R> struct Trig { static constexpr TrigTab<R> v{}; };

template <> __device__ constexpr double ccos<11>(int j) { return Trig<11>::v.c[j]; }
template <> __device__ constexpr double csin<11>(int j) { return Trig<11>::v.s[j]; }
template <> __device__ constexpr double ccos<13>(int j) { return Trig<13>::v.c[j]; }
template <> __device__ constexpr double csin<13>(int j) { return Trig<13>::v.s[j]; }

// In-register DFT of odd length R: U[m] = sum_q u[q] exp(sg 2 pi i q m / R),
// computed from the symmetric and antisymmetric pair sums u[q] +- u[R-q].
template <typename T, int R>
__device__ __forceinline__ void dft(Vt<T> *u, T sg) {
    constexpr int H = (R - 1) / 2;
    Vt<T> sp[H], sm[H];
#pragma unroll
    for (int q = 1; q <= H; ++q) {
        sp[q - 1] = cadd(u[q], u[R - q]);
        sm[q - 1] = csub(u[q], u[R - q]);
    }
    const Vt<T> u0 = u[0];
    Vt<T> tot = u0;
#pragma unroll
    for (int q = 0; q < H; ++q) tot = cadd(tot, sp[q]);
#pragma unroll
    for (int m = 1; m <= H; ++m) {
        Vt<T> a = u0;
        Vt<T> b = mk<T>(T(0), T(0));
#pragma unroll
        for (int q = 1; q <= H; ++q) {
            const int j = (q * m) % R;
            const T cv = T(j <= H ? ccos<R>(j) : ccos<R>(R - j));
            const T sv = T(j <= H ? csin<R>(j) : -csin<R>(R - j));
            a.x += cv * sp[q - 1].x;
            a.y += cv * sp[q - 1].y;
            b.x += sv * sm[q - 1].x;
            b.y += sv * sm[q - 1].y;
        }
        b.x *= sg;
        b.y *= sg;
        u[m] = mk<T>(a.x - b.y, a.y + b.x);
        u[R - m] = mk<T>(a.x + b.y, a.y - b.x);
    }
    u[0] = tot;
}

constexpr int smallest_prime_factor(int n) {
    for (int p = 2; p * p <= n; ++p)
        if (n % p == 0) return p;
    return n;
}

// In-register DFT of length R (any product of 3, 5, 7, 11, 13): prime lengths use the
// symmetric butterflies above, composite ones R = R1 R2 a Cooley-Tukey split
// (R2 DFTs of length R1, twiddles exp(sg 2 pi i n2 k1 / R), R1 DFTs of length
// R2, output index k1 + R1 k2).
template <typename T, int R>
__device__ __forceinline__ void dftn(Vt<T> *u, T sg) {
    if constexpr (R == 3 || R == 5 || R == 7 || R == 11 || R == 13) {
        dft<T, R>(u, sg);
    } else if constexpr (R == 15) {
        // Good-Thomas split 15 = 3 * 5 (coprime, no twiddles): input index
        // (5 n1 + 3 n2) mod 15, output index (10 k1 + 6 k2) mod 15
        Vt<T> y[3][5];
#pragma unroll
        for (int n2 = 0; n2 < 5; ++n2) {
            Vt<T> col[3];
#pragma unroll
            for (int n1 = 0; n1 < 3; ++n1) col[n1] = u[(5 * n1 + 3 * n2) % 15];
            dft<T, 3>(col, sg);
#pragma unroll
            for (int k1 = 0; k1 < 3; ++k1) y[k1][n2] = col[k1];
        }
#pragma unroll
        for (int k1 = 0; k1 < 3; ++k1) {
            dft<T, 5>(y[k1], sg);
#pragma unroll
            for (int k2 = 0; k2 < 5; ++k2) u[(10 * k1 + 6 * k2) % 15] = y[k1][k2];
        }
    } else {
        constexpr int R1 = smallest_prime_factor(R);
        constexpr int R2 = R / R1;
        Vt<T> y[R];
#pragma unroll
        for (int n2 = 0; n2 < R2; ++n2) {
            Vt<T> col[R1];
#pragma unroll
            for (int n1 = 0; n1 < R1; ++n1) col[n1] = u[n1 * R2 + n2];
            dftn<T, R1>(col, sg);
#pragma unroll
            for (int k1 = 0; k1 < R1; ++k1) {
                const int j = (n2 * k1) % R;
                if (j == 0) {
                    y[k1 * R2 + n2] = col[k1];
                } else {
                    const T c = T(Trig<R>::v.c[j]);
                    const T sn = sg * T(Trig<R>::v.s[j]);
                    y[k1 * R2 + n2] = mk<T>(col[k1].x * c - col[k1].y * sn, col[k1].x * sn + col[k1].y * c);
                }
            }
        }
#pragma unroll
        for (int k1 = 0; k1 < R1; ++k1) {
            Vt<T> row[R2];
#pragma unroll
            for (int n2 = 0; n2 < R2; ++n2) row[n2] = y[k1 * R2 + n2];
            dftn<T, R2>(row, sg);
#pragma unroll
            for (int k2 = 0; k2 < R2; ++k2) u[k1 + R1 * k2] = row[k2];
        }
    }
}

// Deterministic work-group sum (fixed shuffle tree, then waves in order) over
// a work-group of at most NT threads; the result is valid in thread 0.
template <int NT>
__device__ double block_sum_t(double v) {
    __shared__ double red[NT / 64];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) red[wave] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0) {
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += red[w];
    }
    __syncthreads();
    return s;
}
__device__ double block_sum(double v) { return block_sum_t<kThreads>(v); }

// K work-group sums at once, each in the order of block_sum (a shuffle tree
// per wave, then the waves in turn), written to out[0 .. K-1] by the first K
// threads: one barrier for all K instead of three per sum.
template <int K>
__device__ void block_sum_many(const double (&v)[K], double *out) {
    __shared__ double red[K][kThreads / 64];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        double x = v[k];
        for (int off = 32; off > 0; off >>= 1) x += __shfl_down(x, off, 64);
        if (lane == 0) red[k][wave] = x;
    }
    __syncthreads();
    if (threadIdx.x < K) {
        double s = 0.0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += red[threadIdx.x][w];
        out[threadIdx.x] = s;
    }
}

__device__ __forceinline__ int wrapi(int i, int L) { return i < (L + 1) / 2 ? i : i - L; }
__device__ __forceinline__ int posmod(int k, int n) {
    int r = k % n;
    return r < 0 ? r + n : r;
}

// Orthonormal basis t_a(k) (a < nc) of the admissible directions at frequency k:
// primal (E_N): k/|k|; dual (J_N), d = 2: R k/|k| with R the rotation by +90
// degrees; d = 3: t1 = k x e_j / |k x e_j| with j the axis of smallest |k_j|
// (lowest index on ties) and t2 = s(k) k/|k| x t1 with s(k) the sign of the
// first non-zero k_j.  Every t_a is odd in k, so a field i sum_a t_a(k) c_a(k)
// is real exactly when each c_a is Hermitian.  Returns 0 at k = 0.
template <typename T>
__device__ __forceinline__ int basis(int d, int kind, int k1, int k2, int k3, T t[2][3]) {
    // straight-line code (selects, no branches): written per branch, the
    // compiler keeps the partially written rows of t on the stack
    // |k|^2 and |k x e_j|^2 are exact integers; rsqrt (reciprocal square
    // root, within a few ulp) replaces a square root and a division, and the
    // second one is only formed for the 3D dual (kind is uniform per launch)
    const T a = T(k1), b = T(k2), c = T(d == 3 ? k3 : 0);
    const T nn = a * a + b * b + c * c;
    const T inv = nn == T(0) ? T(0) : rsqrt(nn);
    const T h1 = a * inv, h2 = b * inv, h3 = c * inv;
    const int ab1 = k1 < 0 ? -k1 : k1, ab2 = k2 < 0 ? -k2 : k2, ab3 = k3 < 0 ? -k3 : k3;
    const bool x1 = ab1 <= ab2 && ab1 <= ab3;  // k x e_1
    const bool x2 = !x1 && ab2 <= ab3;         // k x e_2, else k x e_3
    T u1 = x1 ? T(0) : x2 ? -c : b;
    T u2 = x1 ? c : x2 ? T(0) : -a;
    T u3 = x1 ? -b : x2 ? a : T(0);
    const bool primal = kind == KIND_E, two = d == 2;
    T un = T(0);
    if (!primal && !two) {
        const T uu = u1 * u1 + u2 * u2 + u3 * u3;
        un = uu == T(0) ? T(0) : rsqrt(uu);
    }
    u1 *= un;
    u2 *= un;
    u3 *= un;
    const T s = (k1 != 0) ? (k1 > 0 ? T(1) : T(-1)) : (k2 != 0) ? (k2 > 0 ? T(1) : T(-1)) : (k3 > 0 ? T(1) : T(-1));
    t[0][0] = primal ? h1 : two ? -h2 : u1;
    t[0][1] = primal ? h2 : two ? h1 : u2;
    t[0][2] = primal ? h3 : two ? T(0) : u3;
    t[1][0] = s * (h2 * u3 - h3 * u2);
    t[1][1] = s * (h3 * u1 - h1 * u3);
    t[1][2] = s * (h1 * u2 - h2 * u1);
    return nn == T(0) ? 0 : (primal || two) ? 1 : 2;
}

// 1 / |k| as basis() forms it (0 at k = 0)
template <typename T> __device__ __forceinline__ T inv_norm(int k1, int k2, int k3) {
    const T a = T(k1), b = T(k2), c = T(k3);
    const T nn = a * a + b * b + c * c;
    return nn == T(0) ? T(0) : rsqrt(nn);
}

// exp(-i pi sum_a s_a k_a / N_a) of the shift s (S(s) of Lemma reduce_grid);
// 1 when no shift is set.
__device__ __forceinline__ void shift_phase(const PencilArgs &a, int k1, int k2, int k3, double *c, double *s) {
    const double x = (a.shift[0] ? (double)k1 / a.Nfull[0] : 0.0) + (a.shift[1] ? (double)k2 / a.Nfull[1] : 0.0) +
                     (a.shift[2] ? (double)k3 / a.Nfull[2] : 0.0);
    sincospi(-x, s, c);
}
__device__ __forceinline__ bool has_shift(const PencilArgs &a) { return (a.shift[0] | a.shift[1] | a.shift[2]) != 0; }

__device__ __forceinline__ double sinc_pi(double x) {
    return x == 0.0 ? 1.0 : sinpi(x) / (M_PI * x);
}

// Symmetric material matrix at linear grid point pt from d (d + 1) / 2 fields
// (entries 11, 12, [13,] 22, [23,] 33; field f at g + f * stride).
template <typename T>
__device__ __forceinline__ void sym_load(const T *g, long stride, long pt, int d, T *m) {
    int f = 0;
    for (int i = 0; i < d; ++i)
        for (int j = i; j < d; ++j) {
            const T v = g[(long)f * stride + pt];
            m[i * d + j] = v;
            m[j * d + i] = v;
            ++f;
        }
}

// ---------------------------------------------------------------------------
// Specialised transforms for the grid sizes in kFastSched: compile-time
// schedules with composite radices done in registers (Cooley-Tukey with
// constant internal twiddles), in-place stages staged through registers (one
// LDS buffer), and all d components of a batch transformed together.
// ---------------------------------------------------------------------------
// One in-place Stockham stage over NB transforms of length N: every thread
// first loads all inputs of its butterflies into registers, then (after a
// barrier) twiddles, transforms and stores them.  Column layout (ROWL false)
// with NA < NB: only the NA transforms 0 .. (NA - 1) / 2 and NB - NA / 2 ..
// NB - 1 (the non-zero frequencies of a zero-padded axis) are done.
template <typename T, int R, int N, int P, int NB, bool ROWL, int NT = kThreads, int NA = NB>
__device__ __forceinline__ void stage_ip(Vt<T> *X, const Vt<T> *__restrict__ tw, T sg) {
    constexpr int TQ = N / R;
    constexpr int NT_ = ROWL ? NB : NA;  // transforms done
    constexpr int TOT = TQ * NT_;
    constexpr int PER = (TOT + NT - 1) / NT;
    auto colmap = [](int c) { return c < (NA + 1) / 2 ? c : c + (NB - NA); };
    Vt<T> u[PER][R];
#pragma unroll
    for (int t = 0; t < PER; ++t) {
        const int idx = threadIdx.x + t * NT;
        if (PER * NT == TOT || idx < TOT) {
            const int b = ROWL ? idx / TQ : colmap(idx % NA);
            const int i = ROWL ? idx % TQ : idx / NA;
#pragma unroll
            for (int q = 0; q < R; ++q) {
                const int pos = i + q * TQ;
                u[t][q] = ROWL ? X[b * N + pos] : X[pos * NB + b];
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < PER; ++t) {
        const int idx = threadIdx.x + t * NT;
        if (PER * NT == TOT || idx < TOT) {
            const int b = ROWL ? idx / TQ : colmap(idx % NA);
            const int i = ROWL ? idx % TQ : idx / NA;
            const int k = i % P;
            if constexpr (P > 1) {
#pragma unroll
                for (int q = 1; q < R; ++q) {
                    Vt<T> w = tw[(q - 1) * P + k];
                    w.y *= -sg;
                    u[t][q] = cmul(u[t][q], w);
                }
            }
            dftn<T, R>(u[t], sg);
            const int j = (i - k) * R + k;
#pragma unroll
            for (int q = 0; q < R; ++q) {
                const int pos = j + q * P;
                if (ROWL)
                    X[b * N + pos] = u[t][q];
                else
                    X[pos * NB + b] = u[t][q];
            }
        }
    }
    __syncthreads();
}

template <typename T, int FI, int S, int P, int OFF, int NB, bool ROWL, int NT = kThreads, int NA = NB>
__device__ __forceinline__ void fft_ip(Vt<T> *X, const Vt<T> *tw, T sg) {
    if constexpr (S < kFastSched[FI].nst) {
        constexpr int R = kFastSched[FI].r[S];
        stage_ip<T, R, kFastSched[FI].n, P, NB, ROWL, NT, NA>(X, tw + OFF, sg);
        fft_ip<T, FI, S + 1, P * R, OFF + (R - 1) * P, NB, ROWL, NT, NA>(X, tw, sg);
    }
}


// Copy the n - 1 twiddles of a specialised transform into LDS (read by every
// stage; a global read per butterfly twiddle would stall each stage).
// Only short tables are staged: for n = 2025 the table (32 KB in FP64) would
// cost more occupancy than its reads cost latency.
constexpr bool tw_in_lds(int n, int es) { return n * es <= 12 * 1024; }
constexpr size_t tw_lds_entries(int n, int es) { return tw_in_lds(n, es) ? (size_t)n : 0; }
template <typename T, int N, int NTH = kThreads>
__device__ __forceinline__ const Vt<T> *twiddles_to_lds(Vt<T> *dst, const Vt<T> *__restrict__ src) {
    if constexpr (!tw_in_lds(N, sizeof(Vt<T>))) {
        return src;
    } else {
        for (int i = threadIdx.x; i < N - 1; i += NTH) dst[i] = src[i];
        return dst;
    }
}

// Problem owning this work-group in a multi-problem launch (binary search of
// the work-group offsets); *lb receives the problem-local work-group index.
// Work-groups are dispatched to the 8 XCDs round-robin (physical index mod 8);
// each XCD has its own L2.  Map the physical index to a logical one so that
// every XCD receives a contiguous range of logical tiles: neighbouring tiles
// (which share 128-byte lines of the strided operands) then meet in one L2.
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_logical(int b, int total) {
    const int q = total / kXcds, r = total % kXcds;
    const int x = b % kXcds, k = b / kXcds;
    return x < r ? x * (q + 1) + k : r * (q + 1) + (x - r) * q + k;
}

__device__ __forceinline__ int find_problem(const int *__restrict__ woff, int np, int *lb) {
    int lo = 0, hi = np - 1;
    const int bx = xcd_logical(blockIdx.x, gridDim.x);
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (woff[mid] <= bx)
            lo = mid;
        else
            hi = mid - 1;
    }
    *lb = bx - woff[lo];
    return lo;
}

// Launch target of the specialised kernels: the stream and, for timing, the
// events the dispatch records at its own start and end.
struct Disp {
    hipStream_t s;
    LaunchEv ev;
    Disp(hipStream_t st, LaunchEv e = LaunchEv{}) : s(st), ev(e) {}
};
template <typename... KArgs, typename... Args>
void dispatch(void (*kernel)(KArgs...), dim3 grid, dim3 block, size_t lds, const Disp &d, Args... args) {
    if (d.ev.start != nullptr)
        hipExtLaunchKernelGGL(kernel, grid, block, (std::uint32_t)lds, d.s, d.ev.start, d.ev.stop, 0u, args...);
    else
        hipLaunchKernelGGL(kernel, grid, block, lds, d.s, args...);
}

}  // namespace
}  // namespace fftgal
