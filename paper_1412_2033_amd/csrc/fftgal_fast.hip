// Specialised transform passes of the lengths in kFastSched (compile-time
// schedules): the strided-axis pass, the row passes and the energy Gram.  The
// file is compiled kFastParts times; part FFTGAL_PART holds the lengths whose
// index in kFastSched leaves the remainder FFTGAL_PART modulo kFastParts.
#include "fftgal_device.h"

namespace fftgal {
namespace {

// ---- transforms in LDS: the stages in order, and transposed in reverse order ----
constexpr bool palindromic(int fi) {
    const int s = kFastSched[fi].nst;
    for (int i = 0; i < s; ++i)
        if (kFastSched[fi].r[i] != kFastSched[fi].r[s - 1 - i]) return false;
    return true;
}
constexpr int sched_p(int fi, int st) {
    int p = 1;
    for (int i = 0; i < st; ++i) p *= kFastSched[fi].r[i];
    return p;
}
constexpr int sched_off(int fi, int st) {
    int off = 0, p = 1;
    for (int i = 0; i < st; ++i) {
        off += (kFastSched[fi].r[i] - 1) * p;
        p *= kFastSched[fi].r[i];
    }
    return off;
}
template <typename T, int FI, int S, int SEND, int NB, int NT, bool ROWL = true>
__device__ __forceinline__ void fft_mid(Vt<T> *X, const Vt<T> *tw, T sg) {
    if constexpr (S < SEND) {
        stage_ip<T, kFastSched[FI].r[S], kFastSched[FI].n, sched_p(FI, S), NB, ROWL, NT>(X, tw + sched_off(FI, S), sg);
        fft_mid<T, FI, S + 1, SEND, NB, NT, ROWL>(X, tw, sg);
    }
}

// One in-place stage of the transposed flow: butterfly i reads (i - k) R + k + q P,
// transforms, applies the twiddles and writes i + q N / R.
template <typename T, int R, int N, int P, int NB, int NT, bool ROWL = true>
__device__ __forceinline__ void stage_tr(Vt<T> *X, const Vt<T> *__restrict__ tw, T sg) {
    constexpr int TQ = N / R;
    constexpr int TOT = TQ * NB;
    constexpr int PER = (TOT + NT - 1) / NT;
    Vt<T> u[PER][R];
#pragma unroll
    for (int t = 0; t < PER; ++t) {
        const int idx = threadIdx.x + t * NT;
        if (PER * NT == TOT || idx < TOT) {
            const int b = ROWL ? idx / TQ : idx % NB, i = ROWL ? idx % TQ : idx / NB;
            const int k = i % P;
            const int j = (i - k) * R + k;
#pragma unroll
            for (int q = 0; q < R; ++q) u[t][q] = ROWL ? X[b * N + j + q * P] : X[(j + q * P) * NB + b];
        }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < PER; ++t) {
        const int idx = threadIdx.x + t * NT;
        if (PER * NT == TOT || idx < TOT) {
            const int b = ROWL ? idx / TQ : idx % NB, i = ROWL ? idx % TQ : idx / NB;
            dftn<T, R>(u[t], sg);
            if constexpr (P > 1) {
                const int k = i % P;
#pragma unroll
                for (int q = 1; q < R; ++q) {
                    Vt<T> w = tw[(q - 1) * P + k];
                    w.y *= -sg;
                    u[t][q] = cmul(u[t][q], w);
                }
            }
#pragma unroll
            for (int q = 0; q < R; ++q) {
                if (ROWL)
                    X[b * N + i + q * TQ] = u[t][q];
                else
                    X[(i + q * TQ) * NB + b] = u[t][q];
            }
        }
    }
    __syncthreads();
}

// Stages S .. S1 of the transposed flow, downwards.
template <typename T, int FI, int S, int NB, int NT, int S1 = 0, bool ROWL = true>
__device__ __forceinline__ void fft_tr(Vt<T> *X, const Vt<T> *tw, T sg) {
    if constexpr (S >= S1) {
        stage_tr<T, kFastSched[FI].r[S], kFastSched[FI].n, sched_p(FI, S), NB, NT, ROWL>(X, tw + sched_off(FI, S), sg);
        fft_tr<T, FI, S - 1, NB, NT, S1, ROWL>(X, tw, sg);
    }
}

// ---- Bluestein transforms (FftDesc): NB circular convolutions of length L = N ----
// Convolution lengths with Bluestein kernels: those of the non-smooth transform
// lengths from 11 on.
constexpr bool seven_smooth(int n) {
    for (int p : {3, 5, 7})
        while (n % p == 0) n /= p;
    return n == 1;
}
constexpr bool has_blue(int fi, int d) {
    return seven_smooth(kFastSched[fi].n) && kFastSched[fi].n >= 21 && (d == 2 || kFastSched[fi].n <= kMaxFast3);
}

// The last forward stage, the product with the filter for the sign sg, and
// the first stage of the transposed way back: all on the thread's own points.
template <typename T, int FI, int NB, int NT, bool ROWL>
__device__ __forceinline__ void blue_mid(Vt<T> *X, const Vt<T> *__restrict__ tw, const Vt<T> *__restrict__ H, T sg) {
    constexpr int N = kFastSched[FI].n, S = kFastSched[FI].nst, R = kFastSched[FI].r[S - 1];
    constexpr int TQ = N / R, OFF = sched_off(FI, S - 1);
    constexpr int TOT = TQ * NB;
    for (int idx = threadIdx.x; idx < TOT; idx += NT) {
        const int b = ROWL ? idx / TQ : idx % NB, i = ROWL ? idx % TQ : idx / NB;
        Vt<T> *x = ROWL ? X + b * N + i : X + i * NB + b;
        constexpr int LS = ROWL ? TQ : TQ * NB;
        Vt<T> u[R];
#pragma unroll
        for (int q = 0; q < R; ++q) u[q] = x[q * LS];
#pragma unroll
        for (int q = 1; q < R; ++q) u[q] = cmul(u[q], tw[OFF + (q - 1) * TQ + i]);
        dftn<T, R>(u, T(-1));
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int k = i + q * TQ;  // H_k, or conj(H_{-k}) for sg = -1
            Vt<T> h = H[sg > T(0) || k == 0 ? k : N - k];
            h.y *= sg;
            u[q] = cmul(u[q], h);
        }
        dftn<T, R>(u, T(1));
#pragma unroll
        for (int q = 1; q < R; ++q) {
            Vt<T> w = tw[OFF + (q - 1) * TQ + i];
            w.y = -w.y;
            u[q] = cmul(u[q], w);
        }
#pragma unroll
        for (int q = 0; q < R; ++q) x[q * LS] = u[q];
    }
    __syncthreads();
}

// The convolution of inputs already multiplied by the chirp and padded with
// zeros; the outputs still need the chirp.  S1 > 0 leaves the transposed
// stages below S1 to the caller.
template <typename T, int FI, int NB, int NT, bool ROWL, int S0 = 0, int S1 = 0>
__device__ __forceinline__ void blue_conv(Vt<T> *X, const Vt<T> *tw, const Vt<T> *H, T sg) {
    constexpr int S = kFastSched[FI].nst;
    fft_mid<T, FI, S0, S - 1, NB, NT, ROWL>(X, tw, T(-1));
    blue_mid<T, FI, NB, NT, ROWL>(X, tw, H, sg);
    fft_tr<T, FI, S - 2, NB, NT, S1, ROWL>(X, tw, T(1));
}

// c_m = exp(sg i pi m^2 / n)
template <typename T> __device__ __forceinline__ Vt<T> chirp_at(const Vt<T> *chirp, int m, T sg) {
    Vt<T> c = chirp[m];
    c.y *= sg;
    return c;
}

// row pairs per work-group of the specialised anisotropic row pass so that
// one batch of all d components stays within 24 KB of LDS (the passes are
// latency-bound: smaller work-groups put more of them on a CU)
constexpr bool small_tile(int n, int d);
constexpr int fast_batch(int n, int es, int d) {
    const int cap = 24 * 1024;
    int b = !small_tile(n, d) ? 16 : d == 2 ? 2 : 4;
    while (b > 1 && d * b * n * es > cap) b /= 2;
    return b;
}

// pencils per work-group of the specialised strided-axis pass: one batch of
// all d components within 24 KB of LDS, or 48 KB for 3D FP64 transforms of
// more than 225 points, where the larger batch keeps more of the work-group
// busy in the butterfly stages; elsewhere (2D, shorter 3D transforms) the
// smaller work-groups, more of them per CU, measured faster.  The 3D
// transforms of 225 points (order 113) take tiles sized to the rounds of
// resident work-groups, set by the axis-1 passes and their 113 x 57 pencils:
// in FP32, 9 pencils (50 KB of LDS, three work-groups per CU) make 716
// tiles, one round of the 768 work-groups that fit at once; in FP64 (twice
// the bytes, more than all LDS of the chip holds) 7 pencils (79 KB, two per
// CU) make 921 tiles, under two rounds of 512.  The 2D FP32 transforms of 729
// points (order 365) take 3 pencils with 512 threads (486 of the 2 x 3 x 81
// radix-9 butterflies busy in one round, against two rounds for 2 pencils and
// 256 threads): a batch of 16 such solves 7 % faster.
// Small grids take small tiles, so that their few pencils spread over the CUs:
// in 2D transforms below 330 points one pencil (n / 4 pencils make a pass), in
// 3D up to 63 points two and up to 135 points four.  Per iteration of all 2d
// solves: 2D 189 x 135 FP64 33.3 -> 29.3 us, 2D 315^2 FP32 30.3 -> 27.2, 3D 45^3
// FP32 36.2 -> 29.5; at 405^2 one pencil cost 5 %, at 75^3 two cost 6 %.  Four
// passes of a dual 3D solve, FP32, with the pencils that 24 KB hold (eight, at
// 135 points four) and with four: 75^3 25.2 -> 21.5 us, 105^3 31.2 -> 27.7, 125^3
// 38.3 -> 34.8, 135^3 38.7; FP64 (four, at 135 points two) 135^3 57.1 -> 46.0.
// From 147 points on four were no better in FP32 and 1 % worse at 189^3 FP64.
constexpr bool small_tile(int n, int d) { return d == 2 ? n < 330 : n <= 63; }
constexpr int kFourPencils = 135;  // longest 3D transform that takes four pencils
// Two components of 3D gradient fields.  Schedules of two stages of radix 9 or
// 15 (81, 135, 225 points) take nine pencils and 512 threads: a stage's 18 n / r
// butterflies fill one round of the threads, and two FP64 tiles of 225 points
// fit a CU.  The others take two pencils up to 63 points, four up to 135, then
// what 20 KB hold.  Expand and project together, in us, FP64 / FP32, with the
// pencils 20 KB hold and now: 75^3 13.8 / 15.4 -> 11.9 / 10.6, 81^3 11.5 / 12.9
// -> 11.9 / 10.5, 105^3 14.8 / 14.0 -> 14.9 / 12.4, 135^3 18.9 / 18.8 -> 17.9 /
// 16.1; 225^3 47.0 / 27.5 (four pencils) -> 45.0 / 24.5.  Nine pencils lose where
// a stage takes more rounds or leaves lanes idle: 125^3 16.0 / 14.4 -> 17.4 / 16.3,
// 147^3 FP64 20.5 -> 22.2, 243^3 58.7 / 36.2 -> 79.1 / 38.4.  At order 113 two
// components in place of three took expand / project from 31.4 / 29.4 to 25.9 /
// 23.5 us per launch, FP64.
constexpr bool nine_pencils(int n) {
    const int fi = fast_index(n);
    if (kFastSched[fi].nst != 2) return false;
    for (int i = 0; i < 2; ++i)
        if (kFastSched[fi].r[i] != 9 && kFastSched[fi].r[i] != 15) return false;
    return true;
}
constexpr int two_batch(int n, int es, bool blue) {
    if (!blue && nine_pencils(n)) return 9;
    if (!blue && n <= kFourPencils) return small_tile(n, 3) ? 2 : 4;
    const int cap = blue && n > 105 ? 36 * 1024 : 20 * 1024;
    int b = blue ? 8 : 16;
    while (b > 1 && 2 * b * n * es > cap) b /= 2;
    return b;
}
constexpr int two_nt(int n, bool blue) {
    if (!blue && nine_pencils(n)) return 512;
    return !blue && small_tile(n, 3) ? 128 : kThreads;
}
// Bluestein tiles: up to 8 pencils within 24 KB for the short lengths (their
// grids are small), 48 KB for the others, whose two transforms per pencil need
// the lanes.
// d = 1 stands for the two-component passes of 3D gradient fields.
constexpr int pencil_batch(int n, int es, int d, bool blue = false) {
    if (d == 1) return two_batch(n, es, blue);
    if (blue) {
        const int most = n <= 105 ? 24 * 1024 : 48 * 1024;
        int b = 8;
        while (b > 1 && d * b * n * es > most) b /= 2;
        return b;
    }
    if (d == 3 && n == 225) return es >= 16 ? 7 : 9;
    if (es < 16 && d == 2 && n == 729) return 3;
    if (small_tile(n, d)) return d == 2 ? 1 : 2;
    if (d == 3 && n <= kFourPencils) return 4;
    const int cap = (es >= 16 && d == 3 && n > 225) ? 48 * 1024 : 24 * 1024;
    int b = 16;
    while (b > 1 && d * b * n * es > cap) b /= 2;
    return b;
}

// threads of the specialised strided-axis pass: 512 for the 2D FP64 pencils
// of 2025 points (one pencil of both components per work-group), the 2D FP32
// tiles of 729 points and the 3D tiles of 225 points (315 or 405 transforms of
// 15 points per stage), so that every stage of the transform takes one round
// of the threads; else 256
constexpr int pencil_nt(int n, int es, int d, bool blue = false) {
    if (d == 1) return two_nt(n, blue);
    if (blue) return n >= 1125 ? 512 : kThreads;
    if (small_tile(n, d)) return 128;
    return ((es >= 16 && d == 2 && n >= 2025) || (es < 16 && d == 2 && n == 729) || (d == 3 && n == 225))
               ? 512
               : kThreads;
}

// Bound by memory on large grids (3D, order 113: 4.3 to 4.9 TB/s), on small ones
// by the latency of its loads and stages.  Against the kernel of run-time
// lengths, FP64: 175^3 65 -> 19 us a launch, BLUE 99^3 (through 225) 102 -> 27 us.
//
// BLUE: Bluestein transforms of the length a.f.n through the convolution
// length N; the inputs are multiplied by the chirp on their way into LDS, the
// outputs on their way out.
//
// TWO: EXPAND and PROJECT passes of 3D gradient fields (E_N) in two components.
// The field i k c / |k| has the components 2 and 3 equal to k2 v and k3 v with
// one v = i c / |k|, and k2, k3 are constant along axis 1: between the axis-1
// and axis-2 passes only (i k1 c / |k|, v) are transformed and stored, the axis-2
// inverse pass (a.grad) scales v into its components 2 and 3 as it loads them,
// and the axis-2 forward pass stores k2 y2 + k3 y3 for the projection.  The
// intermediate is a third smaller each way, and so is the axis-1 work.
template <typename T, int FI, int D, bool BLUE, bool TWO>
__global__ __launch_bounds__(pencil_nt(kFastSched[FI].n, sizeof(Vt<T>), TWO ? 1 : D, BLUE))
void pencil_fast(const PencilArgs *__restrict__ pa, const int *__restrict__ woff, int np) {
    using V = Vt<T>;
    constexpr int N = kFastSched[FI].n;
    constexpr int NC = TWO ? 2 : D;  // components transformed
    constexpr int NT = pencil_nt(N, sizeof(V), TWO ? 1 : D, BLUE);
    constexpr int B = pencil_batch(N, sizeof(V), TWO ? 1 : D, BLUE);
    constexpr int NB = NC * B;  // LDS layout [pos][component][batch]
    constexpr int LPI = NT / NB;  // positions per step of the plain prologue / epilogue
    int lb;
    const PencilArgs &a = pa[find_problem(woff, np, &lb)];
    if (a.status != nullptr && a.status->done) return;
    // loads of a starting work-group before the stages of running ones (the
    // priority drops again once the batch is in LDS)
    __builtin_amdgcn_s_setprio(3);
    extern __shared__ __align__(16) unsigned char smem_raw[];  // 16-byte complex doubles
    V *X = reinterpret_cast<V *>(smem_raw);
    const int gx = (a.nb + B - 1) / B;
    const int o = lb / gx;
    const int b0 = (lb - o * gx) * B;
    const int nbw = min(B, a.nb - b0);
    const V *tw = twiddles_to_lds<T, N, NT>(X + N * NB, reinterpret_cast<const V *>(a.tw) + a.f.twoff[0]);
    const T sg = T(a.sgn);
    const T scale = T(a.scale);
    const V zero = mk<T>(T(0), T(0));
    const int n = BLUE ? a.f.n : N;  // transform length
    const V *chirp = reinterpret_cast<const V *>(a.tw) + a.f.choff;
    const V *H = reinterpret_cast<const V *>(a.tw) + a.f.hoff;
    auto place = [&](int k) { return BLUE ? (k < 0 ? k + n : k) : posmod(k, N); };  // position of frequency k
    // pencil b0 + bb sits at (b0 + bb) / Nh, (b0 + bb) % Nh: one division per
    // work-group, then at most one carry per pencil (B <= Nh is not assumed)
    const int q0 = b0 / a.Nh, r0 = b0 - q0 * a.Nh;
    auto split = [&](int bb, int *qb, int *rb) {
        int r = r0 + bb, q = q0;
        while (r >= a.Nh) {
            r -= a.Nh;
            ++q;
        }
        *qb = q;
        *rb = r;
    };
    auto freq = [&](int l, int L, int bb, int *k1, int *k2, int *k3) {
        *k1 = wrapi(l, L);
        int qb, rb;
        split(bb, &qb, &rb);
        if (D == 3) {
            *k2 = wrapi(qb, a.Nmid);
            *k3 = rb;
        } else {
            *k2 = rb;
            *k3 = 0;
        }
    };
    // Global loads of a phase are issued together (branch-free, with idle
    // slots reading an in-range address) into scalar register arrays, then
    // written to LDS.  The input frequencies k in [-(L_in / 2), khi) sit at
    // positions 0 .. khi - 1 and N - L_in / 2 .. N - 1, so the positions
    // khi .. khi + N - L_in - 1 form one contiguous zero band of the LDS batch,
    // written by a loop of its own; slots of idle pencils in the input range
    // are written as zeros by the loading threads.  The trip counts are
    // compile-time bounds: inputs of at most (N + 1) / 2 points (zero-padded
    // transforms) or of N points.
    const int khi = (a.L_in + 1) / 2;
    // zero position z of the N - L_in ones (BLUE: the high input frequencies
    // end at n - 1, and n .. N - 1 are zeros too)
    auto zpos = [&](int z) {
        const int p = khi + z;
        return BLUE && p >= n - (a.L_in - khi) ? p + (a.L_in - khi) : p;
    };
    if (a.pro == PRO_EXPAND) {
      // the CG vectors hold at most (N + 1) / 2 frequencies per axis (Ga), or N
      // (GaNi, transforms on the grid of the approximation order itself)
      auto expand = [&](auto cap) {
        constexpr int PE = (decltype(cap)::value * B + NT - 1) / NT;
        const auto *sr = gbl(reinterpret_cast<const V *>(a.st_r));
        auto *sp = gbl(reinterpret_cast<V *>(a.st_p));
        const auto *sx = gbl(reinterpret_cast<const V *>(a.st_x));
        const T beta = (a.update_p && a.status) ? T(a.status->beta) : T(0);
        T ax[PE][2], ay[PE][2], bx[PE][2], by[PE][2];
#pragma unroll
        for (int t = 0; t < PE; ++t) {
            const int idx = threadIdx.x + t * NT;
            const int bb = idx % B;
            const int l = idx / B;
            const bool ok = idx < a.L_in * B && bb < nbw;
            const long off = ok ? (long)l * a.in_ls + b0 + bb : (long)b0;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const long o2 = (c < a.nc ? c : 0) * a.st_cs + off;
                const V va = a.update_p ? gld(sr + o2) : gld(sx + o2);
                const V vb = a.update_p ? gld(sp + o2) : zero;
                ax[t][c] = va.x;
                ay[t][c] = va.y;
                bx[t][c] = vb.x;
                by[t][c] = vb.y;
            }
        }
        for (int idx = threadIdx.x; idx < (N - a.L_in) * NB; idx += NT) {
            if constexpr (BLUE)
                X[zpos(idx / NB) * NB + idx % NB] = zero;
            else
                X[khi * NB + idx] = zero;
        }
#pragma unroll
        for (int t = 0; t < PE; ++t) {
            const int idx = threadIdx.x + t * NT;
            const int bb = idx % B;
            const int l = idx / B;
            if (idx >= a.L_in * B) continue;
            if (bb >= nbw) {  // idle pencil of a ragged tile
                const int pos = place(wrapi(l, a.L_in));
#pragma unroll
                for (int al = 0; al < NC; ++al) X[pos * NB + al * B + bb] = zero;
                continue;
            }
            int k1, k2, k3;
            freq(l, a.L_in, bb, &k1, &k2, &k3);
            T tb[2][3];
            const int nt = basis<T>(D, a.kind, k1, k2, k3, tb);
            if constexpr (TWO) tb[0][1] = inv_norm<T>(k1, k2, k3);
            V v[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                v[c] = zero;
                if (c < a.nc) {
                    if (a.update_p) {
                        v[c] = mk<T>(ax[t][c] + beta * bx[t][c], ay[t][c] + beta * by[t][c]);
                        gst(sp + c * a.st_cs + (long)l * a.in_ls + b0 + bb, v[c]);
                    } else {
                        v[c] = mk<T>(ax[t][c], ay[t][c]);
                    }
                }
            }
            const int pos = place(k1);
            double pc = 1.0, ps = 0.0;
            if (has_shift(a)) shift_phase(a, k1, k2, k3, &pc, &ps);
#pragma unroll
            for (int al = 0; al < NC; ++al) {
                T ex = T(0), ey = T(0);
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    if (c < nt) {
                        ex -= tb[c][al] * v[c].y;
                        ey += tb[c][al] * v[c].x;
                    }
                }
                if (has_shift(a)) {
                    const T nx = ex * T(pc) - ey * T(ps);
                    ey = ex * T(ps) + ey * T(pc);
                    ex = nx;
                }
                V v1 = mk<T>(ex, ey);
                if constexpr (BLUE) v1 = cmul(v1, chirp_at<T>(chirp, pos, sg));
                X[pos * NB + al * B + bb] = v1;
            }
        }
      };
      if (BLUE || 2 * a.L_in <= N + 1)
          expand(std::integral_constant<int, (N + 1) / 2>{});
      else
          expand(std::integral_constant<int, BLUE ? 1 : N>{});
    } else {
        // every thread owns one LDS slot rr (component c, pencil bb) of LPI
        // positions per step, so its addresses advance by a constant stride;
        // slots of idle pencils in the input range are written as zeros, the
        // zero band outside it by a loop over the band alone
        const int rr = threadIdx.x % NB;
        const int l0 = threadIdx.x / NB;
        const bool act = threadIdx.x < LPI * NB;
        const int c = rr / B;
        const int bb = rr - c * B;
        const bool grad_in = !TWO && D == 3 && a.grad && a.sgn > 0;
        const auto *in = gbl(reinterpret_cast<const V *>(a.in) + (long)o * a.in_os + b0 +
                             (long)(grad_in ? min(c, 1) : c) * a.in_cs + bb);
        auto load = [&](auto cap) {
            constexpr int P = (decltype(cap)::value + LPI - 1) / LPI;
            T vx[P], vy[P];
#pragma unroll
            for (int t = 0; t < P; ++t) {
                const int l = l0 + t * LPI;
                const bool ok = act && l < a.L_in && bb < nbw;
                const V v = gld(in + (ok ? (long)l * a.in_ls : 0L));
                vx[t] = ok ? v.x : T(0);
                vy[t] = ok ? v.y : T(0);
            }
            const int nz = N - a.L_in;  // zero band: positions khi .. khi + nz - 1
            for (int l = l0; act && l < nz; l += LPI) X[zpos(l) * NB + rr] = zero;
#pragma unroll
            for (int t = 0; t < P; ++t) {
                const int l = l0 + t * LPI;
                if (act && l < a.L_in) {
                    const int pos = place(wrapi(l, a.L_in));
                    V v1 = mk<T>(vx[t], vy[t]);
                    if (grad_in && c > 0) {  // component 2: k2 v, component 3: k3 v
                        const T k = T(c == 1 ? wrapi(l, a.L_in) : b0 + bb);
                        v1.x *= k;
                        v1.y *= k;
                    }
                    if constexpr (BLUE) v1 = cmul(v1, chirp_at<T>(chirp, pos, sg));
                    X[pos * NB + rr] = v1;
                }
            }
        };
        if (BLUE || 2 * a.L_in <= N + 1)
            load(std::integral_constant<int, (N + 1) / 2>{});
        else
            load(std::integral_constant<int, BLUE ? 1 : N>{});
    }
    __syncthreads();
    __builtin_amdgcn_s_setprio(0);
    if constexpr (BLUE)
        blue_conv<T, FI, NB, NT, false>(X, tw, H, sg);
    else
        fft_ip<T, FI, 0, 1, 0, NB, false, NT>(X, tw, sg);
    auto *out = gbl(reinterpret_cast<V *>(a.out));
    if (a.epi == EPI_PROJECT) {
      // the projected vector holds at most (N + 1) / 2 frequencies per axis (Ga) or N (GaNi)
      auto project = [&](auto cap) -> double {
        constexpr int PE = (decltype(cap)::value * B + NT - 1) / NT;
        const auto *dv = gbl(reinterpret_cast<const V *>(a.st_dot));
        T dx[PE][2], dy[PE][2];
        if (a.st_dot != nullptr) {
#pragma unroll
            for (int t = 0; t < PE; ++t) {
                const int idx = threadIdx.x + t * NT;
                const int bb = idx % B;
                const int l = idx / B;
                const bool ok = idx < a.L_out * B && bb < nbw;
                const long off = ok ? (long)l * a.out_ls + b0 + bb : (long)b0;
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const V v = gld(dv + (c < a.nc ? c : 0) * a.out_cs + off);
                    dx[t][c] = v.x;
                    dy[t][c] = v.y;
                }
            }
        }
        double part = 0.0;
#pragma unroll
        for (int t = 0; t < PE; ++t) {
            const int idx = threadIdx.x + t * NT;
            const int bb = idx % B;
            const int l = idx / B;
            if (idx >= a.L_out * B || bb >= nbw) continue;
            int k1, k2, k3;
            freq(l, a.L_out, bb, &k1, &k2, &k3);
            T tb[2][3];
            const int nt = basis<T>(D, a.kind, k1, k2, k3, tb);
            if constexpr (TWO) tb[0][1] = inv_norm<T>(k1, k2, k3);
            const int pos = place(k1);
            V y[NC];
#pragma unroll
            for (int al = 0; al < NC; ++al) y[al] = X[pos * NB + al * B + bb];
            if constexpr (BLUE) {
                const V ch = chirp_at<T>(chirp, pos, sg);
#pragma unroll
                for (int al = 0; al < NC; ++al) y[al] = cmul(y[al], ch);
            }
            const double w = (D == 3 ? k3 : k2) == 0 ? 1.0 : 2.0;  // half spectrum: k_d > 0 counts twice
            double pc = 1.0, ps = 0.0;
            if (has_shift(a)) shift_phase(a, k1, k2, k3, &pc, &ps);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                if (c < a.nc) {
                    T qx = T(0), qy = T(0);
                    if (c < nt) {
#pragma unroll
                        for (int al = 0; al < NC; ++al) {
                            const T tt = tb[c][al] * scale;
                            qx += tt * y[al].y;
                            qy -= tt * y[al].x;
                        }
                    }
                    const long off = c * a.out_cs + (long)l * a.out_ls + b0 + bb;
                    if (has_shift(a)) {  // S*(s): the conjugate phase
                        const T nx = qx * T(pc) + qy * T(ps);
                        qy = qy * T(pc) - qx * T(ps);
                        qx = nx;
                    }
                    if (a.accumulate) {
                        const V old = gld(out + off);
                        qx += old.x;
                        qy += old.y;
                    }
                    gst(out + off, mk<T>(qx, qy));
                    if (a.st_dot != nullptr) {
                        part += w * ((double)dx[t][c] * (double)qx + (double)dy[t][c] * (double)qy);
                    } else {
                        part += w * ((double)qx * (double)qx + (double)qy * (double)qy);
                    }
                }
            }
        }
        return part;
      };
      const double part = (BLUE || 2 * a.L_out <= N + 1) ? project(std::integral_constant<int, (N + 1) / 2>{})
                                                         : project(std::integral_constant<int, BLUE ? 1 : N>{});
        const double s = block_sum_t<NT>(part);
        if (threadIdx.x == 0) a.partial[lb] = s;
    } else {
        const int rr = threadIdx.x % NB;
        const int c = rr / B;
        const int bb = rr - c * B;
        const bool grad_out = !TWO && D == 3 && a.grad && a.sgn < 0;
        if (threadIdx.x < LPI * NB && bb < nbw && !(grad_out && c == 2)) {
            auto *ob = out + (long)c * a.out_cs + (long)o * a.out_os + b0 + bb;
            for (int l = threadIdx.x / NB; l < a.L_out; l += LPI) {
                const int pos = place(wrapi(l, a.L_out));
                V v = X[pos * NB + rr];
                if (grad_out && c == 1) {  // k2 y2 + k3 y3
                    const T k2 = T(wrapi(l, a.L_out)), k3 = T(b0 + bb);
                    const V y3 = X[pos * NB + rr + B];
                    v.x = k2 * v.x + k3 * y3.x;
                    v.y = k2 * v.y + k3 * y3.y;
                }
                if constexpr (BLUE) v = cmul(v, chirp_at<T>(chirp, pos, sg));
                v.x *= scale;
                v.y *= scale;
                gst(ob + (long)l * a.out_ls, v);
            }
        }
    }
}

template <typename T, int FI, int D>
__global__ __launch_bounds__(kThreads) void row_fast(const RowArgs *__restrict__ ra, const int *__restrict__ woff,
                                                     int np) {
    using V = Vt<T>;
    constexpr int N = kFastSched[FI].n;
    constexpr int RP = fast_batch(N, sizeof(V), D);
    constexpr int NB = D * RP;  // LDS layout [component][row pair][pos]
    int lb;
    const RowArgs &a = ra[find_problem(woff, np, &lb)];
    if (a.status != nullptr && a.status->done) return;
    extern __shared__ __align__(16) unsigned char smem_raw[];  // 16-byte complex doubles
    V *X = reinterpret_cast<V *>(smem_raw);
    const int nh = a.Nh_row;
    const V *tw = twiddles_to_lds<T, N>(X + N * NB, reinterpret_cast<const V *>(a.tw) + a.f.twoff[0]);
    V *data = reinterpret_cast<V *>(a.data);
    const T *g = reinterpret_cast<const T *>(a.g);
    const int pair0 = lb * RP;
    const int nvp = min(RP, (a.nrows + 1) / 2 - pair0);
    const V zero = mk<T>(T(0), T(0));
    T A0[D * D], Dm[D * D];
#pragma unroll
    for (int i = 0; i < D * D; ++i) {
        A0[i] = T(a.A0[i]);
        Dm[i] = T(a.D[i]);
    }
    // material values of this thread's grid points, loaded before the
    // transforms so that their latency overlaps them
    constexpr int MP = (RP * N + kThreads - 1) / kThreads;
    T gv1[MP], gv2[MP];
#pragma unroll
    for (int t = 0; t < MP; ++t) {
        const int idx = threadIdx.x + t * kThreads;
        const int j = idx / N;
        const int x = idx - j * N;
        gv1[t] = T(0);
        gv2[t] = T(0);
        if (idx < RP * N && j < nvp && a.nfield <= 1) {
            const int r1 = 2 * (pair0 + j);
            gv1[t] = g[(long)r1 * N + x];
            if (r1 + 1 < a.nrows) gv2[t] = g[(long)(r1 + 1) * N + x];
        }
    }
    if (a.mode == ROW_OPER) {
        // both rows of every pair, all loads in flight together (nh <= (N + 1) / 2),
        // then the packed Hermitian extension; the zero band nh <= x <= N - nh
        // is written by a disjoint loop
        constexpr int PLR = (NB * ((N + 1) / 2) + kThreads - 1) / kThreads;
        const auto *dg = gbl(reinterpret_cast<const V *>(a.data));
        T p1x[PLR], p1y[PLR], p2x[PLR], p2y[PLR];
#pragma unroll
        for (int t = 0; t < PLR; ++t) {
            const int idx = threadIdx.x + t * kThreads;
            const int pc = idx / nh;
            const int kx = idx - pc * nh;
            const int c = pc / RP;
            const int j = pc - c * RP;
            const int r1 = 2 * (pair0 + j);
            const bool ok = idx < NB * nh && j < nvp;
            const bool ok2 = ok && r1 + 1 < a.nrows;
            const long off = ok ? (long)c * a.cs + (long)r1 * nh + kx : 0L;
            const V u1 = gld(dg + off);
            const V u2 = gld(dg + (ok2 ? off + nh : off));
            p1x[t] = u1.x;
            p1y[t] = u1.y;
            p2x[t] = ok2 ? u2.x : T(0);
            p2y[t] = ok2 ? u2.y : T(0);
        }
        for (int idx = threadIdx.x; idx < NB * (N - 2 * nh + 1); idx += kThreads) {
            const int pc = idx / (N - 2 * nh + 1);
            X[pc * N + nh + (idx - pc * (N - 2 * nh + 1))] = zero;
        }
#pragma unroll
        for (int t = 0; t < PLR; ++t) {
            const int idx = threadIdx.x + t * kThreads;
            const int pc = idx / nh;
            const int kx = idx - pc * nh;
            if (idx >= NB * nh) continue;
            const V u1 = mk<T>(p1x[t], p1y[t]);
            const V u2 = mk<T>(p2x[t], p2y[t]);
            if (kx == 0) {
                X[pc * N] = mk<T>(u1.x, u2.x);
            } else {
                X[pc * N + kx] = mk<T>(u1.x - u2.y, u1.y + u2.x);
                X[pc * N + N - kx] = mk<T>(u1.x + u2.y, u2.x - u1.y);
            }
        }
        __syncthreads();
        fft_ip<T, FI, 0, 1, 0, NB, true>(X, tw, T(1));
#pragma unroll
        for (int t = 0; t < MP; ++t) {
            const int idx = threadIdx.x + t * kThreads;
            const int j = idx / N;
            const int x = idx - j * N;
            if (idx >= RP * N || j >= nvp) continue;
            V e[D];
#pragma unroll
            for (int b = 0; b < D; ++b) e[b] = X[(b * RP + j) * N + x];
            T m1[D * D], m2[D * D];
            if (a.nfield > 1) {
                const int r1 = 2 * (pair0 + j);
                sym_load<T>(g, a.gstride, (long)r1 * N + x, D, m1);
                if (r1 + 1 < a.nrows)
                    sym_load<T>(g, a.gstride, (long)(r1 + 1) * N + x, D, m2);
                else
#pragma unroll
                    for (int i = 0; i < D * D; ++i) m2[i] = T(0);
            } else {
                const T g1 = gv1[t];
                const T g2 = gv2[t];
#pragma unroll
                for (int i = 0; i < D * D; ++i) {
                    m1[i] = A0[i] + g1 * Dm[i];
                    m2[i] = A0[i] + g2 * Dm[i];
                }
            }
#pragma unroll
            for (int al = 0; al < D; ++al) {
                T y1 = T(0), y2 = T(0);
#pragma unroll
                for (int b = 0; b < D; ++b) {
                    y1 += m1[al * D + b] * e[b].x;
                    y2 += m2[al * D + b] * e[b].y;
                }
                X[(al * RP + j) * N + x] = mk<T>(y1, y2);
            }
        }
    } else {  // ROW_RHS: y = A(x) E on both rows, |y|^2 and y.E partial sums
        double load = 0.0, work = 0.0;
#pragma unroll
        for (int t = 0; t < MP; ++t) {
            const int idx = threadIdx.x + t * kThreads;
            if (idx >= RP * N) continue;
            const int j = idx / N;
            const int x = idx - j * N;
            V y[D];
#pragma unroll
            for (int al = 0; al < D; ++al) y[al] = zero;
            if (j < nvp) {
                const int r1 = 2 * (pair0 + j);
                const int r2 = r1 + 1;
                const bool v2 = r2 < a.nrows;
                T m1[D * D], m2[D * D];
                if (a.nfield > 1) {
                    sym_load<T>(g, a.gstride, (long)r1 * N + x, D, m1);
                    if (v2)
                        sym_load<T>(g, a.gstride, (long)r2 * N + x, D, m2);
                    else
#pragma unroll
                        for (int i = 0; i < D * D; ++i) m2[i] = T(0);
                } else {
                    const T g1 = gv1[t];
                    const T g2 = gv2[t];
#pragma unroll
                    for (int i = 0; i < D * D; ++i) {
                        m1[i] = A0[i] + g1 * Dm[i];
                        m2[i] = A0[i] + g2 * Dm[i];
                    }
                }
#pragma unroll
                for (int al = 0; al < D; ++al) {
                    T y1 = T(0), y2 = T(0);
#pragma unroll
                    for (int b = 0; b < D; ++b) {
                        y1 += m1[al * D + b] * T(a.E[b]);
                        if (v2) y2 += m2[al * D + b] * T(a.E[b]);
                    }
                    y[al] = mk<T>(y1, y2);
                    load += (double)y1 * y1 + (double)y2 * y2;
                    work += ((double)y1 + (double)y2) * a.E[al];
                }
            }
#pragma unroll
            for (int al = 0; al < D; ++al) X[(al * RP + j) * N + x] = y[al];
        }
        const double s = block_sum(load);
        const double s2 = block_sum(work);
        if (threadIdx.x == 0) {
            a.partial[lb] = s;
            if (a.partial2 != nullptr) a.partial2[lb] = s2;
        }
    }
    __syncthreads();
    fft_ip<T, FI, 0, 1, 0, NB, true>(X, tw, T(-1));
    const T half = T(a.scale) * T(0.5);
    for (int idx = threadIdx.x; idx < NB * nh; idx += kThreads) {
        const int pc = idx / nh;
        const int kx = idx - pc * nh;
        const int c = pc / RP;
        const int j = pc - c * RP;
        if (j >= nvp) continue;
        const int r1 = 2 * (pair0 + j);
        const int r2 = r1 + 1;
        const V w = X[pc * N + kx];
        const V wm = X[pc * N + (kx == 0 ? 0 : N - kx)];
        data[(long)c * a.cs + (long)r1 * nh + kx] = mk<T>((w.x + wm.x) * half, (w.y - wm.y) * half);
        if (r2 < a.nrows)
            data[(long)c * a.cs + (long)r2 * nh + kx] = mk<T>((w.y + wm.y) * half, (wm.x - w.x) * half);
    }
}


// ---------------------------------------------------------------------------
// Operator row pass for isotropic materials, A(x) = (a0 + g(x) dA) I.  Every
// component row is multiplied by the same scalar field, so each packed row
// pair (two real rows as one complex transform) is independent of the others.
// The first inverse stage reads its points straight from the half-spectrum
// rows (Hermitian extension and zero padding on the fly); the last inverse
// stage leaves each thread holding the points x = i + q N/R, where the
// material multiply is applied and the first forward stage (same radix, same
// points) follows in registers.  Only the middle stages, the exchanges
// between stages and the final Hermitian unpacking go through LDS.
// transforms per work-group and work-group size: every thread of the first
// and last stages owns one butterfly of radix r[0]
constexpr int iso_tb(int fi) {
    const int tq = kFastSched[fi].n / kFastSched[fi].r[0];
    // transforms of more than 128 butterflies per stage (n = 2025): one per
    // work-group, so that several share a CU
    return tq <= 64 ? 128 / tq : (tq <= 128 ? 256 / tq : 1);
}
constexpr int iso_nt(int fi) {
    const int tq = kFastSched[fi].n / kFastSched[fi].r[0];
    return (iso_tb(fi) * tq + 63) / 64 * 64;
}

constexpr bool has_iso(int fi) { return fi < kNumGridLengths && palindromic(fi); }
constexpr bool has_staged(int fi) { return has_iso(fi) && kFastSched[fi].nst == 2; }
constexpr size_t pencil_lds(int n, int es, int d, bool blue = false) {
    return (size_t)es * ((size_t)n * (d == 1 ? 2 : d) * pencil_batch(n, es, d, blue) + tw_lds_entries(n, es));
}
constexpr size_t row_lds(int n, int es, int d) {
    return (size_t)es * ((size_t)n * d * fast_batch(n, es, d) + tw_lds_entries(n, es));
}
template <typename T> constexpr size_t iso_lds(int fi) {
    const int n = kFastSched[fi].n;
    if (kFastSched[fi].nst == 2) return sizeof(T) * (size_t)iso_tb(fi) * n + sizeof(Vt<T>) * n;
    return sizeof(Vt<T>) * ((size_t)iso_tb(fi) * n + tw_lds_entries(n, sizeof(Vt<T>)));
}

template <typename T, int FI>
__global__ __launch_bounds__(iso_nt(FI)) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 3 : 1)))
void row_iso_fast(const RowArgs *__restrict__ ra,
                                                           const int *__restrict__ woff, int np) {
    using V = Vt<T>;
    constexpr int N = kFastSched[FI].n;
    constexpr int S = kFastSched[FI].nst;
    constexpr int R = kFastSched[FI].r[0];
    constexpr int TQ = N / R;  // butterflies per transform in the first and last stages
    constexpr int TB = iso_tb(FI);
    constexpr int NT = iso_nt(FI);
    constexpr int OFFL = sched_off(FI, S - 1);  // twiddles of the last stage (P = TQ)
    static_assert(palindromic(FI) && S >= 2 && sched_p(FI, S - 1) == TQ, "schedule must be palindromic");
    int lb;
    const RowArgs &a = ra[find_problem(woff, np, &lb)];
    if (a.status != nullptr && a.status->done) return;
    extern __shared__ __align__(16) unsigned char smem_raw[];  // 16-byte complex doubles
    V *X = reinterpret_cast<V *>(smem_raw);  // [transform][pos]
    // stage twiddles staged in LDS when short; for the longest rows (2025
    // points, 32 KB in FP64) the LDS goes to the transforms and the twiddles
    // are read through the cache
    const V *twg = reinterpret_cast<const V *>(a.tw) + a.f.twoff[0];
    const V *tws = twiddles_to_lds<T, N, NT>(X + TB * N, twg);
    const V zero = mk<T>(T(0), T(0));
    const int nh = a.Nh_row;
    const int npairs = (a.nrows + 1) / 2;
    const int ntr = a.d * npairs;
    const int tl = threadIdx.x / TQ;
    const int i = threadIdx.x - tl * TQ;
    const int tb = lb * TB + tl;
    const bool act = tl < TB && tb < ntr;
    // transforms ordered pair-major (components fastest), so that the d
    // transforms reading one row pair's material values share a work-group
    int c = 0, r1 = 0;
    if (act) {
        const int pr = tb / a.d;
        c = tb - pr * a.d;
        r1 = 2 * pr;
    }
    const bool v2 = act && r1 + 1 < a.nrows;
    const V *data = reinterpret_cast<const V *>(a.data);
    const V *row1 = data + (long)c * a.cs + (long)r1 * nh;
    const T *g = reinterpret_cast<const T *>(a.g);
    const T a0 = T(a.A0[0]);
    const T da = T(a.D[0]);
    V u[R];
    {
        // all loads first (idle points read entry 0 of the pair), then the
        // Hermitian packing by selects
        T l1x[R], l1y[R], l2x[R], l2y[R];
        const auto *rg = gbl(row1);
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int pos = i + q * TQ;
            const int kx = pos < nh ? pos : (pos > N - nh ? N - pos : 0);
            const V a1 = gld(rg + kx);
            const V a2 = gld(rg + (v2 ? nh + kx : kx));
            l1x[q] = a1.x;
            l1y[q] = a1.y;
            l2x[q] = a2.x;
            l2y[q] = a2.y;
        }
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int pos = i + q * TQ;
            const V u1 = mk<T>(l1x[q], l1y[q]);
            const V u2 = v2 ? mk<T>(l2x[q], l2y[q]) : zero;
            const V lo = pos == 0 ? mk<T>(u1.x, u2.x) : mk<T>(u1.x - u2.y, u1.y + u2.x);
            const V hi = mk<T>(u1.x + u2.y, u2.x - u1.y);
            u[q] = !act ? zero : (pos < nh ? lo : (pos > N - nh ? hi : zero));
        }
    }
    // first inverse stage (P = 1): outputs at i R + q
    dftn<T, R>(u, T(1));
    if (act) {
#pragma unroll
        for (int q = 0; q < R; ++q) X[tl * N + i * R + q] = u[q];
    }
    __syncthreads();
    fft_mid<T, FI, 1, S - 1, TB, NT>(X, tws, T(1));
    // last inverse stage: inputs and outputs at i + q TQ (own points only)
    if (act) {
#pragma unroll
        for (int q = 0; q < R; ++q) u[q] = X[tl * N + i + q * TQ];
    }
    __syncthreads();
#pragma unroll
    for (int q = 1; q < R; ++q) {
        V w = tws[OFFL + (q - 1) * TQ + i];
        w.y = -w.y;
        u[q] = cmul(u[q], w);
    }
    dftn<T, R>(u, T(1));
    // the two real rows at x = i + q TQ: multiply by a0 + g da (the material
    // values are loaded here, not held through the inverse stages; idle lanes
    // read row r1, in range, and their products are never stored)
    {
        const T *gr1 = g + (long)r1 * N + i;
        const T *gr2 = v2 ? gr1 + N : gr1;
        T g1[R], g2[R];
#pragma unroll
        for (int q = 0; q < R; ++q) {
            g1[q] = gr1[q * TQ];
            g2[q] = gr2[q * TQ];
        }
#pragma unroll
        for (int q = 0; q < R; ++q) {
            u[q].x *= a0 + g1[q] * da;
            u[q].y *= a0 + g2[q] * da;
        }
    }
    // first forward stage on the same points
    dftn<T, R>(u, T(-1));
    if (act) {
#pragma unroll
        for (int q = 0; q < R; ++q) X[tl * N + i * R + q] = u[q];
    }
    __syncthreads();
    fft_mid<T, FI, 1, S - 1, TB, NT>(X, tws, T(-1));
    if (act) {
#pragma unroll
        for (int q = 0; q < R; ++q) u[q] = X[tl * N + i + q * TQ];
#pragma unroll
        for (int q = 1; q < R; ++q) u[q] = cmul(u[q], tws[OFFL + (q - 1) * TQ + i]);
        dftn<T, R>(u, T(-1));
#pragma unroll
        for (int q = 0; q < R; ++q) X[tl * N + i + q * TQ] = u[q];
    }
    __syncthreads();
    // unpack the two rows of each transform and keep the first nh frequencies
    V *out = reinterpret_cast<V *>(a.data);
    const T half = T(a.scale) * T(0.5);
    for (int o = threadIdx.x; o < TB * nh; o += NT) {
        const int t = o / nh;
        const int kx = o - t * nh;
        const int tbo = lb * TB + t;
        if (tbo >= ntr) continue;
        const int po = tbo / a.d;
        const int co = tbo - po * a.d;
        const int ro = 2 * po;
        const V w = X[t * N + kx];
        const V wm = X[t * N + (kx == 0 ? 0 : N - kx)];
        V *orow = out + (long)co * a.cs + (long)ro * nh;
        orow[kx] = mk<T>((w.x + wm.x) * half, (w.y - wm.y) * half);
        if (ro + 1 < a.nrows) orow[nh + kx] = mk<T>((w.y + wm.y) * half, (wm.x - w.x) * half);
    }
}

// Variant for two-stage schedules: every exchange between stages moves the
// real parts through LDS first and the imaginary parts second, so a transform
// needs n reals of LDS instead of n complex values; with the material values
// loaded at the multiply (not held in registers) this raises the resident
// waves, which hides the latencies of the stages, and each thread unpacks its
// own points (no index division).
constexpr int split_tb(int fi) { return iso_tb(fi); }
constexpr int split_nt(int fi) { return iso_nt(fi); }

template <typename T, int FI>
__global__ __launch_bounds__(split_nt(FI)) void row_iso_split(const RowArgs *__restrict__ ra,
                                                             const int *__restrict__ woff, int np) {
    using V = Vt<T>;
    constexpr int N = kFastSched[FI].n;
    constexpr int R = kFastSched[FI].r[0];
    constexpr int TQ = N / R;
    constexpr int TB = split_tb(FI);
    constexpr int NT = split_nt(FI);
    constexpr int OFFL = sched_off(FI, 1);
    static_assert(kFastSched[FI].nst == 2 && kFastSched[FI].r[1] == R, "two-stage palindromic schedule");
    int lb;
    const RowArgs &a = ra[find_problem(woff, np, &lb)];
    if (a.status != nullptr && a.status->done) return;
    extern __shared__ __align__(16) unsigned char smem_raw[];  // 16-byte complex doubles
    T *Bf = reinterpret_cast<T *>(smem_raw);            // [transform][pos], one part at a time
    V *tws = reinterpret_cast<V *>(Bf + TB * N);        // last-stage twiddles
    const V *twg = reinterpret_cast<const V *>(a.tw) + a.f.twoff[0];
    for (int i = threadIdx.x; i < N - 1; i += NT) tws[i] = twg[i];
    const V zero = mk<T>(T(0), T(0));
    const int nh = a.Nh_row;
    const int npairs = (a.nrows + 1) / 2;
    const int ntr = a.d * npairs;
    const int tl = threadIdx.x / TQ;
    const int i = threadIdx.x - tl * TQ;
    const int tb = lb * TB + tl;
    const bool act = tl < TB && tb < ntr;
    int c = 0, r1 = 0;
    if (act) {
        const int pr = tb / a.d;
        c = tb - pr * a.d;
        r1 = 2 * pr;
    }
    const bool v2 = act && r1 + 1 < a.nrows;
    V *data = reinterpret_cast<V *>(a.data);
    V *row1 = data + (long)c * a.cs + (long)r1 * nh;
    V *row2 = row1 + nh;
    const T *g = reinterpret_cast<const T *>(a.g);
    T *Bt = Bf + (act ? tl : 0) * N;
    // exchange: write own values at positions wp(q), read positions rp(q)
    auto xchg = [&](V *u, auto wp, auto rp) {
#pragma unroll
        for (int q = 0; q < R; ++q)
            if (act) Bt[wp(q)] = u[q].x;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < R; ++q)
            if (act) u[q].x = Bt[rp(q)];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < R; ++q)
            if (act) Bt[wp(q)] = u[q].y;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < R; ++q)
            if (act) u[q].y = Bt[rp(q)];
        __syncthreads();
    };
    auto stage_out = [&](int q) { return i * R + q; };
    auto own = [&](int q) { return i + q * TQ; };
    V u[R];
    {
        // loads in two groups (idle points read entry 0 of the pair), each
        // followed by the Hermitian packing by selects; the empty asm
        // statements keep the second group from being hoisted, which bounds
        // the registers the staged values need
        const auto *rg = gbl(row1);
        constexpr int LG = (R + 1) / 2;
#pragma unroll
        for (int q0 = 0; q0 < R; q0 += LG) {
            asm volatile("" ::: "memory");
            T l1x[LG], l1y[LG], l2x[LG], l2y[LG];
#pragma unroll
            for (int q = q0; q < q0 + LG && q < R; ++q) {
                const int pos = i + q * TQ;
                const int kx = pos < nh ? pos : (pos > N - nh ? N - pos : 0);
                const V a1 = gld(rg + kx);
                const V a2 = gld(rg + (v2 ? nh + kx : kx));
                l1x[q - q0] = a1.x;
                l1y[q - q0] = a1.y;
                l2x[q - q0] = a2.x;
                l2y[q - q0] = a2.y;
            }
#pragma unroll
            for (int q = q0; q < q0 + LG && q < R; ++q) {
                const int pos = i + q * TQ;
                const V u1 = mk<T>(l1x[q - q0], l1y[q - q0]);
                const V u2 = v2 ? mk<T>(l2x[q - q0], l2y[q - q0]) : zero;
                const V lo = pos == 0 ? mk<T>(u1.x, u2.x) : mk<T>(u1.x - u2.y, u1.y + u2.x);
                const V hi = mk<T>(u1.x + u2.y, u2.x - u1.y);
                u[q] = !act ? zero : (pos < nh ? lo : (pos > N - nh ? hi : zero));
            }
        }
        asm volatile("" ::: "memory");
    }
    dftn<T, R>(u, T(1));
    xchg(u, stage_out, own);
#pragma unroll
    for (int q = 1; q < R; ++q) {
        V w = tws[OFFL + (q - 1) * TQ + i];
        w.y = -w.y;
        u[q] = cmul(u[q], w);
    }
    dftn<T, R>(u, T(1));
    {
        // material values in groups of five loads, issued only here (the
        // empty asm statements keep the compiler from hoisting them over
        // the transform, where they would hold registers)
        const T a0 = T(a.A0[0]);
        const T da = T(a.D[0]);
        const T *g1 = g + (long)r1 * N + i;
        const T *g2 = v2 ? g1 + N : g1;
        constexpr int GQ = 5;
#pragma unroll
        for (int q0 = 0; q0 < R; q0 += GQ) {
            asm volatile("" ::: "memory");
#pragma unroll
            for (int q = q0; q < q0 + GQ && q < R; ++q) {
                const T ga = g1[q * TQ];
                const T gb = g2[q * TQ];
                u[q].x *= a0 + ga * da;
                u[q].y *= a0 + gb * da;
            }
        }
        asm volatile("" ::: "memory");
    }
    dftn<T, R>(u, T(-1));
    xchg(u, stage_out, own);
#pragma unroll
    for (int q = 1; q < R; ++q) u[q] = cmul(u[q], tws[OFFL + (q - 1) * TQ + i]);
    dftn<T, R>(u, T(-1));
    // Hermitian unpacking: each thread pairs its points p < nh with N - p
    // (nh <= (N + 1) / 2, so only the first QH of its points are kept)
    constexpr int QH = ((N + 1) / 2 + TQ - 1) / TQ;
    V m[QH];
    auto partner = [&](int q) {
        const int p = i + q * TQ;
        return p == 0 ? 0 : N - p;
    };
#pragma unroll
    for (int q = 0; q < R; ++q)
        if (act) Bt[own(q)] = u[q].x;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < QH; ++q)
        if (act) m[q].x = Bt[partner(q)];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < R; ++q)
        if (act) Bt[own(q)] = u[q].y;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < QH; ++q)
        if (act) m[q].y = Bt[partner(q)];
    const T half = T(a.scale) * T(0.5);
#pragma unroll
    for (int q = 0; q < QH; ++q) {
        const int p = i + q * TQ;
        if (act && p < nh) {
            const V w = u[q];
            const V wm = m[q];
            row1[p] = mk<T>((w.x + wm.x) * half, (w.y - wm.y) * half);
            if (v2) row2[p] = mk<T>((w.y + wm.y) * half, (wm.x - w.x) * half);
        }
    }
}

// Variant for the row lengths of Ga plans (half-spectrum rows of at most
// (N + 3) / 4 points: order (N + 1) / 2 on the grid N).  Every global load of
// a work-group -- its half-spectrum rows, the material rows of its pairs and
// the last-stage twiddles -- is issued at once and parked in LDS, so a
// work-group waits for memory once.  Work-groups own whole row pairs (all D
// components of each, pair-major), so each material row is fetched once.
// Lanes beyond the last transform repeat the work of the last one, and the
// spare lane of a 16-lane group that of the group's 15th (same inputs, same
// instructions, so their LDS writes store the values already there) instead
// of branching around every LDS access; only the final stores are guarded.
// The transform is that of row_iso_split; per-transform LDS rows are padded
// so that the stride exchanges of neighbouring transforms fall into
// different banks.
constexpr int staged_nhc(int n) { return (n + 3) / 4; }
// lanes per transform: 15 butterflies get an aligned group of 16 lanes (the
// last lane repeats the 15th), so that the lanes of one LDS access pass belong
// to whole transforms
constexpr int staged_lg(int fi) {
    const int tq = kFastSched[fi].n / kFastSched[fi].r[0];
    return tq == 15 ? 16 : tq;
}
// threads per work-group: the best lane utilisation of 128, 192 or 256, except
// for the 3D FP64 rows of 225 points (es: bytes of a complex value), which
// take 256 (five row pairs, three work-groups per CU): 2 % faster than the
// 192 of the best utilisation, while in FP32 the two were alike
constexpr int staged_nt(int fi, int d, int es) {
    if (es >= 16 && d == 3 && kFastSched[fi].n == 225) return 256;
    const int tq = kFastSched[fi].n / kFastSched[fi].r[0];
    int best = 128, bu = 0;  // utilisation in 1/1024
    for (int nt = 128; nt <= 256; nt += 64) {
        const int tb = (nt / staged_lg(fi)) / d * d;
        const int u = tb * tq * 1024 / nt;
        if (u > bu) {
            bu = u;
            best = nt;
        }
    }
    return best;
}
constexpr int staged_tb(int fi, int d, int es) { return (staged_nt(fi, d, es) / staged_lg(fi)) / d * d; }
// LDS row stride of one transform (in reals): 240 = 16 (mod 32) for n = 225
constexpr int staged_stride(int fi) { return kFastSched[fi].n == 225 ? 240 : kFastSched[fi].n; }
// twiddles of the second stage: w_n^(q i) at (q - 1) n / r + i (1 <= q < r,
// 0 <= i < n / r), so that the lanes of a transform read consecutive entries
constexpr int staged_ntp(int fi) { return (kFastSched[fi].r[0] - 1) * (kFastSched[fi].n / kFastSched[fi].r[0]); }
template <typename T>
constexpr size_t staged_lds(int fi, int d) {
    const int n = kFastSched[fi].n, tb = staged_tb(fi, d, (int)sizeof(Vt<T>));
    const size_t work = std::max(sizeof(Vt<T>) * tb * 2 * (staged_nhc(n) + 1), sizeof(T) * tb * staged_stride(fi));
    const size_t gm = sizeof(T) * (tb / d) * 2 * n;
    return (gm + 15) / 16 * 16 + sizeof(Vt<T>) * staged_ntp(fi) + work;
}

// three waves per SIMD: what the LDS of four 192-thread or three 256-thread
// work-groups per CU allows in FP64
template <typename T, int FI, int D>
__global__ __launch_bounds__(staged_nt(FI, D, sizeof(Vt<T>))) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 3 : 1)))
void row_iso_staged(const RowArgs *__restrict__ ra,
                                                                  const int *__restrict__ woff, int np) {
    using V = Vt<T>;
    constexpr int N = kFastSched[FI].n;
    constexpr int R = kFastSched[FI].r[0];
    constexpr int TQ = N / R;
    constexpr int TB = staged_tb(FI, D, sizeof(Vt<T>));
    constexpr int PW = TB / D;  // row pairs per work-group
    constexpr int NT = staged_nt(FI, D, sizeof(Vt<T>));
    constexpr int NHC = staged_nhc(N);
    constexpr int SR = NHC + 1;  // staged row: NHC points and a zero slot
    constexpr int S = staged_stride(FI);
    constexpr int NTP = staged_ntp(FI);
    constexpr int OFFL = sched_off(FI, 1);
    constexpr int LG = staged_lg(FI);
    static_assert(kFastSched[FI].nst == 2 && kFastSched[FI].r[1] == R, "two-stage palindromic schedule");
    static_assert(TB * LG <= NT && TB % D == 0 && NT - TB * LG <= LG && LG >= TQ, "work-group shape");
    int lb;
    const RowArgs &a = ra[find_problem(woff, np, &lb)];
    if (a.status != nullptr && a.status->done) return;
    extern __shared__ __align__(16) unsigned char smem_raw[];  // 16-byte complex doubles
    T *Gs = reinterpret_cast<T *>(smem_raw);                                           // [2 PW][N] material
    V *tp = reinterpret_cast<V *>(smem_raw + (sizeof(T) * PW * 2 * N + 15) / 16 * 16);  // [NTP] stage twiddles
    V *St = tp + NTP;                      // [D][2 PW][SR] staged half-spectrum rows ...
    T *Bf = reinterpret_cast<T *>(St);     // ... later [TB][S], one part at a time
    const int nh = a.Nh_row;
    const int npairs = (a.nrows + 1) / 2;
    const int pr0 = lb * PW;
    const int npr = min(PW, npairs - pr0);
    const int nrow_wg = min(2 * npr, a.nrows - 2 * pr0);  // rows of this work-group
    // ---- all global loads in flight together, then parked in LDS; the waves
    // of a work-group issuing its loads take priority over those already in
    // the transform arithmetic, so that a new work-group's loads leave early
    __builtin_amdgcn_s_setprio(3);
    constexpr int GP = (PW * 2 * N + NT - 1) / NT;
    constexpr int RS = 2 * PW * SR;  // staged slots of one component: its 2 PW rows
    constexpr int SPC = (RS + NT - 1) / NT;
    constexpr int NW = (R - 1) * TQ;  // stage-1 twiddles
    constexpr int WP = (NW + NT - 1) / NT;
    const auto *gsrc = gbl(reinterpret_cast<const T *>(a.g) + (long)2 * pr0 * N);
    const auto *dsrc = gbl(reinterpret_cast<const V *>(a.data));
    const auto *twg = gbl(reinterpret_cast<const V *>(a.tw) + a.f.twoff[0] + OFFL);
    const int gcnt = nrow_wg * N;
    T gv[GP];
    T sx[D][SPC], sy[D][SPC];
    T wx[WP], wy[WP];
#pragma unroll
    for (int t = 0; t < GP; ++t) {
        const int idx = threadIdx.x + t * NT;
        gv[t] = gsrc[idx < gcnt ? idx : 0];
    }
    // the rows of a work-group are contiguous in each component: one flat
    // copy per component into slots [c][row][SR] (slot k >= nh and rows past
    // the last are zero), with the offsets of a component in 32 bits
#pragma unroll
    for (int c = 0; c < D; ++c) {
        const auto *dc = dsrc + (long)c * a.cs + (long)2 * pr0 * nh;
#pragma unroll
        for (int t = 0; t < SPC; ++t) {
            const int f = threadIdx.x + t * NT;
            const int row = f / SR;
            const int k = f - row * SR;
            const bool ok = f < RS && k < nh && row < nrow_wg;
            const V v = gld(dc + (ok ? row * nh + k : 0));
            sx[c][t] = ok ? v.x : T(0);
            sy[c][t] = ok ? v.y : T(0);
        }
    }
#pragma unroll
    for (int t = 0; t < WP; ++t) {
        const int idx = threadIdx.x + t * NT;
        const V v = gld(twg + (idx < NW ? idx : 0));
        wx[t] = v.x;
        wy[t] = v.y;
    }
#pragma unroll
    for (int t = 0; t < GP; ++t) {
        const int idx = threadIdx.x + t * NT;
        if (idx < PW * 2 * N) Gs[idx] = idx < gcnt ? gv[t] : T(0);
    }
#pragma unroll
    for (int c = 0; c < D; ++c) {
#pragma unroll
        for (int t = 0; t < SPC; ++t) {
            const int f = threadIdx.x + t * NT;
            if (f < RS) St[c * RS + f] = mk<T>(sx[c][t], sy[c][t]);
        }
    }
#pragma unroll
    for (int t = 0; t < WP; ++t) {
        const int idx = threadIdx.x + t * NT;
        if (idx < NW) tp[idx] = mk<T>(wx[t], wy[t]);
    }
    __syncthreads();
    __builtin_amdgcn_s_setprio(0);
    // ---- packed Hermitian extension of the two rows of this thread's transform
    const int tr = threadIdx.x / LG;
    const int lane = threadIdx.x - tr * LG;
    const int tl = tr < TB ? tr : TB - 1;  // lanes past the last transform repeat it
    const int i = lane < TQ ? lane : TQ - 1;  // and spare lanes of a group repeat its last
    const int lp = tl / D;                 // pair within the work-group
    const int c = tl - lp * D;             // component
    const bool owner = tr < TB && lane < TQ && lp < npr;
    // Points i + q TQ of this thread that lie in the zero band for every
    // thread (NHC <= q TQ and q TQ + TQ - 1 <= N - NHC) are zero on input and
    // not needed on output: with the band known at compile time the compiler
    // drops their arithmetic from the first inverse and the last forward stage.
    auto zband = [](int q) { return q * TQ >= NHC && q * TQ + TQ - 1 <= N - NHC; };
    V u[R];
    {
        const V *s1 = St + c * RS + 2 * lp * SR;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            if (zband(q)) {
                u[q] = mk<T>(T(0), T(0));
                continue;
            }
            // z = u1 + i u2 at p < nh, conj(u1) + i conj(u2) at p > N - nh,
            // (u1.x, u2.x) at p = 0, zero between (the zero slot)
            const int pos = i + q * TQ;
            const bool low = pos < nh;
            const int kx = low ? pos : (pos > N - nh ? N - pos : NHC);
            const V u1 = s1[kx];
            const V u2 = s1[SR + kx];
            const T sg = low ? (pos == 0 ? T(0) : T(1)) : T(-1);
            u[q] = mk<T>(u1.x - sg * u2.y, u2.x + sg * u1.y);
        }
    }
    __syncthreads();  // St is reused as Bf
    T *Bt = Bf + tl * S;
    auto xchg = [&](V *w, auto wp, auto rp) {
#pragma unroll
        for (int q = 0; q < R; ++q) Bt[wp(q)] = w[q].x;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < R; ++q) w[q].x = Bt[rp(q)];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < R; ++q) Bt[wp(q)] = w[q].y;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < R; ++q) w[q].y = Bt[rp(q)];
        __syncthreads();
    };
    auto stage_out = [&](int q) { return i * R + q; };
    auto own = [&](int q) { return i + q * TQ; };
    dftn<T, R>(u, T(1));
    xchg(u, stage_out, own);
#pragma unroll
    for (int q = 1; q < R; ++q) {
        V w = tp[(q - 1) * TQ + i];
        w.y = -w.y;
        u[q] = cmul(u[q], w);
    }
    dftn<T, R>(u, T(1));
    {
        const T a0 = T(a.A0[0]);
        const T da = T(a.D[0]);
        const T *g1 = Gs + 2 * lp * N + i;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            u[q].x *= a0 + g1[q * TQ] * da;
            u[q].y *= a0 + g1[N + q * TQ] * da;
        }
    }
    dftn<T, R>(u, T(-1));
    xchg(u, stage_out, own);
#pragma unroll
    for (int q = 1; q < R; ++q) u[q] = cmul(u[q], tp[(q - 1) * TQ + i]);
    dftn<T, R>(u, T(-1));
    // Hermitian unpacking: outputs p < nh <= NHC pair with N - p > N - NHC,
    // so only the points that can lie there go through LDS
    constexpr int QH = (NHC + TQ - 1) / TQ;
    V m[QH];
    auto partner = [&](int q) {
        const int p = i + q * TQ;
        return p == 0 ? 0 : N - p;
    };
    auto high = [](int q) { return q * TQ + TQ - 1 > N - NHC; };
#pragma unroll
    for (int q = 0; q < R; ++q)
        if (high(q)) Bt[own(q)] = u[q].x;
    Bt[own(0)] = u[0].x;  // p = 0 pairs with itself
    __syncthreads();
#pragma unroll
    for (int q = 0; q < QH; ++q) m[q].x = Bt[partner(q)];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < R; ++q)
        if (high(q)) Bt[own(q)] = u[q].y;
    Bt[own(0)] = u[0].y;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < QH; ++q) m[q].y = Bt[partner(q)];
    if (!owner) return;
    const int r1 = 2 * (pr0 + lp);
    const bool v2 = 2 * lp + 1 < nrow_wg;
    auto *row1 = gbl(reinterpret_cast<V *>(a.data) + (long)c * a.cs + (long)r1 * nh);
    const T half = T(a.scale) * T(0.5);
#pragma unroll
    for (int q = 0; q < QH; ++q) {
        const int p = i + q * TQ;
        if (p < nh) {
            const V w = u[q];
            const V wm = m[q];
            gst(row1 + p, mk<T>((w.x + wm.x) * half, (w.y - wm.y) * half));
            if (v2) gst(row1 + nh + p, mk<T>((w.y + wm.y) * half, (wm.x - w.x) * half));
        }
    }
}

// Energy Gram quadrature (ROW_GRAM) for the specialised lengths: all d^2
// component fields of the d solutions are transformed to the grid in one
// in-place batch, then (A_M (E_s + e_s), E_t + e_t) is summed over the rows.
// Row pairs per work-group: one batch within 48 KB of LDS, so that several
// work-groups share a CU (a single pair of 225-point rows of 9 fields takes
// 32 KB in FP64: four work-groups per CU).
constexpr int gram_batch(int n, int es, int d) {
    int b = 8;
    while (b > 1 && d * d * b * n * es > 48 * 1024) b /= 2;
    return b;
}
constexpr size_t gram_lds(int n, int d) { return (size_t)16 * n * d * d * gram_batch(n, 16, d); }

template <typename T, int FI, int D>
__global__ __launch_bounds__(kThreads) void row_gram_fast(const RowArgs *__restrict__ ra, const int *__restrict__ woff,
                                                          int np) {
    using V = Vt<T>;
    constexpr int N = kFastSched[FI].n;
    constexpr int RP = gram_batch(N, sizeof(V), D);
    constexpr int NC = D * D;
    constexpr int NB = NC * RP;  // LDS layout [component][row pair][pos]
    int lb;
    const RowArgs &a = ra[find_problem(woff, np, &lb)];
    extern __shared__ __align__(16) unsigned char smem_raw[];  // 16-byte complex doubles
    V *X = reinterpret_cast<V *>(smem_raw);
    const int nh = a.Nh_row;
    const V *tw = reinterpret_cast<const V *>(a.tw) + a.f.twoff[0];
    const V *data = reinterpret_cast<const V *>(a.data);
    const T *g = reinterpret_cast<const T *>(a.g);
    const int pair0 = lb * RP;
    const int nvp = min(RP, (a.nrows + 1) / 2 - pair0);
    const V zero = mk<T>(T(0), T(0));
    // every global load of the work-group in flight at once: the half-spectrum
    // rows (at most (N + 1) / 2 points each) and, for the scalar-field form,
    // the material values of the accumulation below; the band of positions
    // no load writes is zeroed by a loop of its own
    constexpr int NHMAX = (N + 1) / 2;
    constexpr int PE = (NB * NHMAX + kThreads - 1) / kThreads;
    constexpr int GP = (RP * N + kThreads - 1) / kThreads;
    V u1v[PE], u2v[PE];
#pragma unroll
    for (int t = 0; t < PE; ++t) {
        const int idx = threadIdx.x + t * kThreads;
        const int pc = idx / nh;
        const int kx = idx - pc * nh;
        const int c = pc / RP;
        const int j = pc - c * RP;
        const bool ok = idx < NB * nh && j < nvp;
        const int r1 = 2 * (pair0 + (ok ? j : 0));
        const bool two = ok && r1 + 1 < a.nrows;
        const long o1 = ok ? (long)c * a.cs + (long)r1 * nh + kx : 0L;
        const long o2 = two ? o1 + nh : 0L;  // in range even if the load is issued
        u1v[t] = ok ? data[o1] : zero;
        u2v[t] = two ? data[o2] : zero;
    }
    T gv1[GP], gv2[GP];
    const bool gpre = a.nfield == 1;
#pragma unroll
    for (int t = 0; t < GP; ++t) {
        const int idx = threadIdx.x + t * kThreads;
        const int j = idx / N;
        const int x = idx - j * N;
        const bool ok = gpre && idx < RP * N && j < nvp;
        const bool two = ok && 2 * (pair0 + j) + 1 < a.nrows;
        const long r1 = 2 * (pair0 + (ok ? j : 0));
        const long i1 = ok ? r1 * N + x : 0L, i2 = two ? i1 + N : 0L;
        gv1[t] = ok ? g[i1] : T(0);
        gv2[t] = two ? g[i2] : T(0);
    }
    const int nzb = N - 2 * nh + 1;  // positions nh .. N - nh of every field
    for (int idx = threadIdx.x; idx < NB * nzb; idx += kThreads) {
        const int pc = idx / nzb;
        X[pc * N + nh + (idx - pc * nzb)] = zero;
    }
#pragma unroll
    for (int t = 0; t < PE; ++t) {
        const int idx = threadIdx.x + t * kThreads;
        if (idx >= NB * nh) continue;
        const int pc = idx / nh;
        const int kx = idx - pc * nh;
        const V u1 = u1v[t], u2 = u2v[t];  // zero for idle row pairs
        if (kx == 0) {
            X[pc * N] = mk<T>(u1.x, u2.x);
        } else {
            X[pc * N + kx] = mk<T>(u1.x - u2.y, u1.y + u2.x);
            X[pc * N + N - kx] = mk<T>(u1.x + u2.y, u2.x - u1.y);
        }
    }
    __syncthreads();
    fft_ip<T, FI, 0, 1, 0, NB, true>(X, tw, T(1));
    T A0[D * D], Dm[D * D];
#pragma unroll
    for (int i = 0; i < D * D; ++i) {
        A0[i] = T(a.A0[i]);
        Dm[i] = T(a.D[i]);
    }
    double gs[D * D];
#pragma unroll
    for (int i = 0; i < D * D; ++i) gs[i] = 0.0;
#pragma unroll
    for (int t = 0; t < GP; ++t) {
        const int idx = threadIdx.x + t * kThreads;
        if (idx >= RP * N) continue;
        const int j = idx / N;
        const int x = idx - j * N;
        if (j >= nvp) continue;
        const int r1 = 2 * (pair0 + j);
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int r = r1 + half;
            if (r >= a.nrows) continue;
            T am[D * D];
            if (a.nfield > 1) {
                sym_load<T>(g, a.gstride, (long)r * N + x, D, am);
            } else {
                const T gg = half ? gv2[t] : gv1[t];
#pragma unroll
                for (int i = 0; i < D * D; ++i) am[i] = A0[i] + gg * Dm[i];
            }
            T f[D][D];
#pragma unroll
            for (int sol = 0; sol < D; ++sol)
#pragma unroll
                for (int b = 0; b < D; ++b) {
                    const V zv = X[((sol * D + b) * RP + j) * N + x];
                    f[sol][b] = (half ? zv.y : zv.x) + (sol == b ? T(1) : T(0));
                }
#pragma unroll
            for (int t = 0; t < D; ++t) {
                T af[D];
#pragma unroll
                for (int al = 0; al < D; ++al) {
                    T y = T(0);
#pragma unroll
                    for (int b = 0; b < D; ++b) y += am[al * D + b] * f[t][b];
                    af[al] = y;
                }
#pragma unroll
                for (int sol = 0; sol < D; ++sol) {
                    T dot = T(0);
#pragma unroll
                    for (int al = 0; al < D; ++al) dot += f[sol][al] * af[al];
                    gs[sol * D + t] += dot;
                }
            }
        }
    }
    block_sum_many<D * D>(gs, a.partial + (long)lb * D * D);
}

// Row pass of an isotropic material, A(x) = (a0 + g(x) dA) I, for any schedule.
// A work-group owns PW row pairs with all D components: D PW transforms of two
// packed real rows in LDS.  Its global loads (half-spectrum rows, material
// rows) are issued together; the inverse stages run in place; the last one
// stays in registers, where the values are multiplied by the material, and the
// first forward stage follows on the same points.  The forward transform is
// the transpose of the inverse flow (the DFT matrix is symmetric): its stages
// run in reverse order, each reading the positions its inverse twin wrote,
// with the twiddles of the same table after the butterfly, so that no stage
// between the two transforms needs an exchange, whatever the radices.  Rows
// whose D transforms would take more than 16 KB run one transform per
// work-group (pair-major, material values read at the multiply), so that
// several work-groups share a CU.  It is bound by memory on large grids and by
// its LDS stages on small ones: 175^3 FP64 50 us a launch (164 MB, 3.3 TB/s), against
// 138 us in the kernel of run-time lengths.
constexpr bool pairs_one(int n, int es, int d) { return d * n * es > 16 * 1024; }
constexpr int pairs_pw(int n, int es, int d) {
    const int cap = 20 * 1024;
    int p = d == 3 ? 4 : n < 330 ? 1 : 2;
    while (p > 1 && d * p * n * es > cap) --p;
    return p;
}
// The first six lengths keep the kernels above.  Theirs -> this one, us: 2025
// points FP64 258 -> 269 and 729 points 43.2 -> 45.6 per iteration of four solves
// at once (2D); 125 points, 3D order 63, the row pass 30.5 -> 29.6 (FP32 17.5 ->
// 15.5), but six solves at once 375 -> 372 (FP32 323 -> 325).  245 points would
// gain: 2D 21.1 -> 20.0 per iteration of four solves, the row pass of 3D order
// 123 155 -> 145 (FP32 71.8 -> 69.9).
constexpr bool has_pairs(int fi) { return fi >= kNumGridLengths; }
constexpr int pairs_tb(int n, int es, int d) { return pairs_one(n, es, d) ? 1 : d * pairs_pw(n, es, d); }
constexpr int pairs_rl(int fi) { return kFastSched[fi].r[kFastSched[fi].nst - 1]; }
constexpr int pairs_nt(int fi, int es, int d) {
    const int n = kFastSched[fi].n, t = pairs_tb(n, es, d) * (n / pairs_rl(fi));
    const int nt = (t + 63) / 64 * 64;
    return nt < 64 ? 64 : nt > 256 ? 256 : nt;
}
constexpr size_t pairs_lds(int fi, int es, int d) {
    const int n = kFastSched[fi].n;
    const size_t g = pairs_one(n, es, d) ? 0 : ((size_t)es * pairs_pw(n, es, d) * n + 15) / 16 * 16;
    return (size_t)es * n * pairs_tb(n, es, d) + es * tw_lds_entries(n, es) + g;
}

template <typename T, int FI, int D>
__global__ __launch_bounds__(pairs_nt(FI, sizeof(Vt<T>), D))
void row_iso_pairs(const RowArgs *__restrict__ ra, const int *__restrict__ woff, int np) {
    using V = Vt<T>;
    constexpr int N = kFastSched[FI].n;
    constexpr int S = kFastSched[FI].nst;
    constexpr int R = pairs_rl(FI);
    constexpr int TQ = N / R;
    constexpr bool ONE = pairs_one(N, sizeof(V), D);
    constexpr int PW = ONE ? 1 : pairs_pw(N, sizeof(V), D);
    constexpr int TB = pairs_tb(N, sizeof(V), D);  // transforms: component c0 + c of pair p is c PW + p
    constexpr int NT = pairs_nt(FI, sizeof(V), D);
    constexpr int OFFL = sched_off(FI, S - 1);
    int lb;
    const RowArgs &a = ra[find_problem(woff, np, &lb)];
    if (a.status != nullptr && a.status->done) return;
    __builtin_amdgcn_s_setprio(3);
    extern __shared__ __align__(16) unsigned char smem_raw[];  // 16-byte complex doubles
    V *X = reinterpret_cast<V *>(smem_raw);
    V *tws = X + TB * N;
    T *Gs = reinterpret_cast<T *>(tws + tw_lds_entries(N, sizeof(V)));  // [2 PW][N] material rows
    const int nh = a.Nh_row;
    const int pr0 = ONE ? lb / D : lb * PW;
    const int c0 = ONE ? lb - pr0 * D : 0;
    const int nrow_wg = min(2 * PW, a.nrows - 2 * pr0);  // rows of this work-group
    constexpr int GP = ONE ? 1 : (2 * PW * N + NT - 1) / NT;
    const auto *gsrc = gbl(reinterpret_cast<const T *>(a.g) + (long)2 * pr0 * N);
    const auto *data = gbl(reinterpret_cast<const V *>(a.data) + (long)c0 * a.cs + (long)2 * pr0 * nh);
    const int gcnt = nrow_wg * N;
    T gv[GP];
#pragma unroll
    for (int t = 0; t < GP && !ONE; ++t) {
        const int idx = threadIdx.x + t * NT;
        gv[t] = gsrc[idx < gcnt ? idx : 0];
    }
    // rows: at most (N + 3) / 4 points (Ga) or (N + 1) / 2 (the grid of the
    // approximation order); idle slots read entry 0 of the work-group's rows
    auto load = [&](auto cap) {
        constexpr int NHC = decltype(cap)::value;
        constexpr int PL = (TB * NHC + NT - 1) / NT;
        T x1[PL], y1[PL], x2[PL], y2[PL];
#pragma unroll
        for (int t = 0; t < PL; ++t) {
            const int idx = threadIdx.x + t * NT;
            const int tr = idx / NHC, k = idx % NHC;
            const int c = tr / PW, p = tr % PW;
            const bool ok = idx < TB * NHC && k < nh && 2 * p < nrow_wg;
            const bool ok2 = ok && 2 * p + 1 < nrow_wg;
            const long off = ok ? (long)c * a.cs + 2 * p * nh + k : 0L;
            const V u1 = gld(data + off);
            const V u2 = gld(data + (ok2 ? off + nh : off));
            x1[t] = ok ? u1.x : T(0);
            y1[t] = ok ? u1.y : T(0);
            x2[t] = ok2 ? u2.x : T(0);
            y2[t] = ok2 ? u2.y : T(0);
        }
        const V *twg = reinterpret_cast<const V *>(a.tw) + a.f.twoff[0];
        const V *tl = twiddles_to_lds<T, N, NT>(tws, twg);
#pragma unroll
        for (int t = 0; t < GP && !ONE; ++t) {
            const int idx = threadIdx.x + t * NT;
            if (idx < 2 * PW * N) Gs[idx] = idx < gcnt ? gv[t] : T(0);
        }
        // zero band nh .. N - nh of every transform
        const int nz = N - 2 * nh + 1;
        for (int idx = threadIdx.x; idx < TB * nz; idx += NT) {
            const int tr = idx / nz;
            X[tr * N + nh + (idx - tr * nz)] = mk<T>(T(0), T(0));
        }
#pragma unroll
        for (int t = 0; t < PL; ++t) {
            const int idx = threadIdx.x + t * NT;
            const int tr = idx / NHC, k = idx % NHC;
            if (idx >= TB * NHC || k >= nh) continue;
            V *xr = X + tr * N;
            if (k == 0) {
                xr[0] = mk<T>(x1[t], x2[t]);
            } else {
                xr[k] = mk<T>(x1[t] - y2[t], y1[t] + x2[t]);
                xr[N - k] = mk<T>(x1[t] + y2[t], x2[t] - y1[t]);
            }
        }
        return tl;
    };
    const bool ga = nh <= staged_nhc(N);
    const V *tw = ga ? load(std::integral_constant<int, staged_nhc(N)>{})
                     : load(std::integral_constant<int, (N + 1) / 2>{});
    __syncthreads();
    __builtin_amdgcn_s_setprio(0);
    fft_mid<T, FI, 0, S - 1, TB, NT>(X, tw, T(1));
    {
        constexpr int TOT = TQ * TB;
        constexpr int PER = (TOT + NT - 1) / NT;
        const T a0 = T(a.A0[0]);
        const T da = T(a.D[0]);
#pragma unroll
        for (int t = 0; t < PER; ++t) {
            const int idx = threadIdx.x + t * NT;
            if (PER * NT != TOT && idx >= TOT) continue;
            const int tr = idx / TQ, i = idx % TQ;
            V *xr = X + tr * N + i;
            T g1[R], g2[R];
            if constexpr (ONE) {  // a missing second row repeats the first (its product is not stored)
                const auto *gp = gsrc + i;
                const auto *gq = nrow_wg > 1 ? gp + N : gp;
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    g1[q] = gp[q * TQ];
                    g2[q] = gq[q * TQ];
                }
            }
            V u[R];
#pragma unroll
            for (int q = 0; q < R; ++q) u[q] = xr[q * TQ];
#pragma unroll
            for (int q = 1; q < R; ++q) {
                V w = tw[OFFL + (q - 1) * TQ + i];
                w.y = -w.y;
                u[q] = cmul(u[q], w);
            }
            dftn<T, R>(u, T(1));
            if constexpr (!ONE) {
                const T *gs = Gs + 2 * (tr % PW) * N + i;
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    g1[q] = gs[q * TQ];
                    g2[q] = gs[N + q * TQ];
                }
            }
#pragma unroll
            for (int q = 0; q < R; ++q) {
                u[q].x *= a0 + g1[q] * da;
                u[q].y *= a0 + g2[q] * da;
            }
            dftn<T, R>(u, T(-1));
#pragma unroll
            for (int q = 1; q < R; ++q) u[q] = cmul(u[q], tw[OFFL + (q - 1) * TQ + i]);
#pragma unroll
            for (int q = 0; q < R; ++q) xr[q * TQ] = u[q];
        }
        __syncthreads();
    }
    fft_tr<T, FI, S - 2, TB, NT>(X, tw, T(-1));
    const T half = T(a.scale) * T(0.5);
    auto *out = gbl(reinterpret_cast<V *>(a.data) + (long)c0 * a.cs + (long)2 * pr0 * nh);
    auto store = [&](auto cap) {
        constexpr int NHC = decltype(cap)::value;
        for (int idx = threadIdx.x; idx < TB * NHC; idx += NT) {
            const int tr = idx / NHC, k = idx % NHC;
            const int c = tr / PW, p = tr % PW;
            if (k >= nh || 2 * p >= nrow_wg) continue;
            const V w = X[tr * N + k];
            const V wm = X[tr * N + (k == 0 ? 0 : N - k)];
            auto *o = out + (long)c * a.cs + 2 * p * nh + k;
            gst(o, mk<T>((w.x + wm.x) * half, (w.y - wm.y) * half));
            if (2 * p + 1 < nrow_wg) gst(o + nh, mk<T>((w.y + wm.y) * half, (wm.x - w.x) * half));
        }
    };
    if (ga)
        store(std::integral_constant<int, staged_nhc(N)>{});
    else
        store(std::integral_constant<int, (N + 1) / 2>{});
}

// Axis 2, rows and back to axis 2 of an isotropic material on small 3D grids
// with equal axes 2 and 3.  A work-group owns one plane x1: the inverse
// transforms along axis 2 of its three half-spectrum fields, the row transforms
// and the material as in row_iso_pairs, and the forward transforms along axis 2,
// all in LDS, so that the plane is read and written once (in place).  On these
// grids each pass takes 6 to 9 us whatever its work (launch, argument and first
// load latency), so one pass in place of three is what counts.
//
// Taken up to 63 points per axis; us per iteration, all six solves at once /
// one solve: 9^3 FP64 22 / 19 -> 18 / 16, 35^3 40 / 35 -> 31 / 27, 45^3 46 / 36
// -> 39 / 31, 63^3 69 / 37 -> 60 / 34, FP32 48 / 29 -> 39 / 26.  From 75 points
// the three passes are as fast or faster: 75^3 FP64 131 / 43 -> 137 / 46, 75^3
// FP32 89 / 36 -> 85 / 39, 105^3 FP32 142 / 45 -> 141 / 43.
// 512 threads within 128 registers let two work-groups share a CU where the LDS
// does (FP64: up to 49 points, 60 KB; 63 points take 98 KB, one per CU); at 45
// points, FP64, 640 and 1024 threads took 44 us (one per CU), 384 took 40.
constexpr int plane_nt(int n) { return n <= 25 ? 256 : 512; }
constexpr size_t plane_lds(int n, int es) {
    return (size_t)es * ((size_t)n * 3 * ((n + 1) / 2) + tw_lds_entries(n, es));
}
constexpr bool has_plane(int n) { return seven_smooth(n) && n <= 63; }

template <typename T, int FI>
__global__ __launch_bounds__(plane_nt(kFastSched[FI].n), 4)
void plane_iso(const RowArgs *__restrict__ ra, const int *__restrict__ woff, int np) {
    using V = Vt<T>;
    constexpr int N = kFastSched[FI].n;
    constexpr int S = kFastSched[FI].nst;
    constexpr int R = pairs_rl(FI);
    constexpr int TQ = N / R;
    constexpr int NT = plane_nt(N);
    constexpr int H = (N + 1) / 2;         // frequencies along axis 2, row pairs
    constexpr int NHC = staged_nhc(N);     // frequencies along axis 3
    constexpr int NB = 3 * NHC;            // axis-2 transforms, LDS layout [pos][component][k3]
    constexpr int TB = 3 * H;              // row pair transforms, LDS layout [component][pair][pos]
    constexpr int OFFL = sched_off(FI, S - 1);
    int lb;
    const RowArgs &a = ra[find_problem(woff, np, &lb)];
    if (a.status != nullptr && a.status->done) return;
    extern __shared__ __align__(16) unsigned char smem_raw[];  // 16-byte complex doubles
    V *X = reinterpret_cast<V *>(smem_raw);
    const int nh = a.Nh_row, L2 = a.L2;
    auto *data = gbl(reinterpret_cast<V *>(a.data) + (long)lb * L2 * nh);
    const auto *gsrc = gbl(reinterpret_cast<const T *>(a.g) + (long)lb * N * N);
    const V zero = mk<T>(T(0), T(0));
    constexpr int PI = (3 * H * NHC + NT - 1) / NT;
    {
        T vx[PI], vy[PI];
#pragma unroll
        for (int t = 0; t < PI; ++t) {
            const int idx = threadIdx.x + t * NT;
            const int k = idx % NHC, l = idx / NHC % H, c = idx / (NHC * H);
            const bool ok = c < 3 && l < L2 && k < nh;
            const V v = gld(data + (ok ? c * a.cs + l * nh + k : 0L));
            vx[t] = ok ? v.x : T(0);
            vy[t] = ok ? v.y : T(0);
        }
        const int khi = (L2 + 1) / 2;
        for (int idx = threadIdx.x; idx < (N - L2) * NB; idx += NT) X[khi * NB + idx] = zero;
#pragma unroll
        for (int t = 0; t < PI; ++t) {
            const int idx = threadIdx.x + t * NT;
            const int k = idx % NHC, l = idx / NHC % H, c = idx / (NHC * H);
            if (c < 3 && l < L2) X[posmod(wrapi(l, L2), N) * NB + c * NHC + k] = mk<T>(vx[t], vy[t]);
        }
    }
    const V *tw = twiddles_to_lds<T, N, NT>(X + N * TB, reinterpret_cast<const V *>(a.tw) + a.f.twoff[0]);
    __syncthreads();
    fft_ip<T, FI, 0, 1, 0, NB, false, NT>(X, tw, T(1));
    constexpr int PL = (TB * NHC + NT - 1) / NT;
    {  // two rows of a pair as one complex row
        V u1[PL], u2[PL];
#pragma unroll
        for (int t = 0; t < PL; ++t) {
            const int idx = threadIdx.x + t * NT;
            const int tr = idx / NHC, k = idx % NHC;
            const int c = tr / H, x2 = 2 * (tr % H);
            u1[t] = u2[t] = zero;
            if (idx < TB * NHC) {
                u1[t] = X[x2 * NB + c * NHC + k];
                if (x2 + 1 < N) u2[t] = X[(x2 + 1) * NB + c * NHC + k];
            }
        }
        __syncthreads();
        const int nz = N - 2 * nh + 1;  // zero band nh .. N - nh of every row
        for (int idx = threadIdx.x; idx < TB * nz; idx += NT) {
            const int tr = idx / nz;
            X[tr * N + nh + (idx - tr * nz)] = zero;
        }
#pragma unroll
        for (int t = 0; t < PL; ++t) {
            const int idx = threadIdx.x + t * NT;
            const int tr = idx / NHC, k = idx % NHC;
            if (idx >= TB * NHC || k >= nh) continue;
            V *xr = X + tr * N;
            if (k == 0) {
                xr[0] = mk<T>(u1[t].x, u2[t].x);
            } else {
                xr[k] = mk<T>(u1[t].x - u2[t].y, u1[t].y + u2[t].x);
                xr[N - k] = mk<T>(u1[t].x + u2[t].y, u2[t].x - u1[t].y);
            }
        }
    }
    __syncthreads();
    fft_mid<T, FI, 0, S - 1, TB, NT>(X, tw, T(1));
    {
        const T a0 = T(a.A0[0]);
        const T da = T(a.D[0]);
        for (int idx = threadIdx.x; idx < TQ * TB; idx += NT) {
            const int tr = idx / TQ, i = idx % TQ;
            const int x2 = 2 * (tr % H);
            V *xr = X + tr * N + i;
            const auto *gp = gsrc + x2 * N + i;
            const auto *gq = x2 + 1 < N ? gp + N : gp;  // a missing second row repeats the first
            T g1[R], g2[R];
#pragma unroll
            for (int q = 0; q < R; ++q) {
                g1[q] = gp[q * TQ];
                g2[q] = gq[q * TQ];
            }
            V u[R];
#pragma unroll
            for (int q = 0; q < R; ++q) u[q] = xr[q * TQ];
#pragma unroll
            for (int q = 1; q < R; ++q) {
                V w = tw[OFFL + (q - 1) * TQ + i];
                w.y = -w.y;
                u[q] = cmul(u[q], w);
            }
            dftn<T, R>(u, T(1));
#pragma unroll
            for (int q = 0; q < R; ++q) {
                u[q].x *= a0 + g1[q] * da;
                u[q].y *= a0 + g2[q] * da;
            }
            dftn<T, R>(u, T(-1));
#pragma unroll
            for (int q = 1; q < R; ++q) u[q] = cmul(u[q], tw[OFFL + (q - 1) * TQ + i]);
#pragma unroll
            for (int q = 0; q < R; ++q) xr[q * TQ] = u[q];
        }
    }
    __syncthreads();
    fft_tr<T, FI, S - 2, TB, NT>(X, tw, T(-1));
    {  // the half spectra of both rows of a pair
        const T half = T(a.scale) * T(0.5);
        V w[PL], wm[PL];
#pragma unroll
        for (int t = 0; t < PL; ++t) {
            const int idx = threadIdx.x + t * NT;
            const int tr = idx / NHC, k = idx % NHC;
            w[t] = wm[t] = zero;
            if (idx < TB * NHC) {
                w[t] = X[tr * N + k];
                wm[t] = X[tr * N + (k == 0 ? 0 : N - k)];
            }
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < PL; ++t) {
            const int idx = threadIdx.x + t * NT;
            const int tr = idx / NHC, k = idx % NHC;
            const int c = tr / H, x2 = 2 * (tr % H);
            if (idx >= TB * NHC) continue;
            V *x = X + x2 * NB + c * NHC + k;
            x[0] = mk<T>((w[t].x + wm[t].x) * half, (w[t].y - wm[t].y) * half);
            if (x2 + 1 < N) x[NB] = mk<T>((w[t].y + wm[t].y) * half, (wm[t].x - w[t].x) * half);
        }
    }
    __syncthreads();
    fft_ip<T, FI, 0, 1, 0, NB, false, NT>(X, tw, T(-1));
#pragma unroll
    for (int t = 0; t < PI; ++t) {
        const int idx = threadIdx.x + t * NT;
        const int k = idx % NHC, l = idx / NHC % H, c = idx / (NHC * H);
        if (c < 3 && l < L2 && k < nh)
            gst(data + (c * a.cs + l * nh + k), X[posmod(wrapi(l, L2), N) * NB + c * NHC + k]);
    }
}

// Row pass of an isotropic material with Bluestein transforms (rows of any
// length n = a.f.n <= (N + 1) / 2): as row_iso_pairs, with each transform a
// convolution of length N.  Between the inverse and the forward transform the
// last transposed stage leaves a thread the points i + q N / R0, where the
// chirp of the one, the material and the chirp of the other multiply the n
// points of the row (the rest is zero padding) and the first stage of the
// forward convolution follows on the same points.
// It is bound by its two convolutions' stages: one pair of 225 FP64 points, 64
// threads, takes 46.6 us at order 99, two pairs and 128 threads 50.6, the kernel
// of run-time lengths took 157.
constexpr int blue_pw(int n, int es, int d) {
    int p = d == 3 ? 4 : 2;
    while (p > 1 && d * p * n * es > 18 * 1024) --p;
    return p;
}
constexpr bool blue_one(int n, int es, int d) { return d * n * es > 24 * 1024; }
constexpr int blue_tb(int n, int es, int d) { return blue_one(n, es, d) ? 1 : d * blue_pw(n, es, d); }
constexpr int blue_nt(int fi, int es, int d) {
    const int n = kFastSched[fi].n, t = blue_tb(n, es, d) * (n / kFastSched[fi].r[0]);
    const int nt = t / 64 * 64 > t * 3 / 4 ? t / 64 * 64 : (t + 63) / 64 * 64;
    return nt < 64 ? 64 : nt > 256 ? 256 : nt;
}
constexpr size_t blue_lds(int fi, int es, int d) {
    const int n = kFastSched[fi].n;
    return (size_t)es * ((size_t)n * blue_tb(n, es, d) + tw_lds_entries(n, es));
}

template <typename T, int FI, int D>
__global__ __launch_bounds__(blue_nt(FI, sizeof(Vt<T>), D))
void row_iso_blue(const RowArgs *__restrict__ ra, const int *__restrict__ woff, int np) {
    using V = Vt<T>;
    constexpr int N = kFastSched[FI].n;
    constexpr int R = kFastSched[FI].r[0];
    constexpr int TQ = N / R;
    constexpr bool ONE = blue_one(N, sizeof(V), D);
    constexpr int PW = ONE ? 1 : blue_pw(N, sizeof(V), D);
    constexpr int TB = blue_tb(N, sizeof(V), D);  // transforms: component c0 + c of pair p is c PW + p
    constexpr int NT = blue_nt(FI, sizeof(V), D);
    constexpr int NHC = ((N + 1) / 2 + 1) / 2;  // stored points of a row of at most (N + 1) / 2
    int lb;
    const RowArgs &a = ra[find_problem(woff, np, &lb)];
    if (a.status != nullptr && a.status->done) return;
    __builtin_amdgcn_s_setprio(3);
    extern __shared__ __align__(16) unsigned char smem_raw[];  // 16-byte complex doubles
    V *X = reinterpret_cast<V *>(smem_raw);
    const int n = a.f.n;
    const int nh = a.Nh_row;
    const int pr0 = ONE ? lb / D : lb * PW;
    const int c0 = ONE ? lb - pr0 * D : 0;
    const int nrow_wg = min(2 * PW, a.nrows - 2 * pr0);  // rows of this work-group
    const V *tab = reinterpret_cast<const V *>(a.tw);
    const V *chirp = tab + a.f.choff;
    const V *H = tab + a.f.hoff;
    auto *data = gbl(reinterpret_cast<V *>(a.data) + (long)c0 * a.cs + (long)2 * pr0 * nh);
    constexpr int PL = (TB * NHC + NT - 1) / NT;
    T x1[PL], y1[PL], x2[PL], y2[PL];
#pragma unroll
    for (int t = 0; t < PL; ++t) {
        const int idx = threadIdx.x + t * NT;
        const int tr = idx / NHC, k = idx % NHC;
        const int c = tr / PW, p = tr % PW;
        const bool ok = idx < TB * NHC && k < nh && 2 * p < nrow_wg;
        const bool ok2 = ok && 2 * p + 1 < nrow_wg;
        const long off = ok ? (long)c * a.cs + 2 * p * nh + k : 0L;
        const V u1 = gld(data + off);
        const V u2 = gld(data + (ok2 ? off + nh : off));
        x1[t] = ok ? u1.x : T(0);
        y1[t] = ok ? u1.y : T(0);
        x2[t] = ok2 ? u2.x : T(0);
        y2[t] = ok2 ? u2.y : T(0);
    }
    const V *tw = twiddles_to_lds<T, N, NT>(X + TB * N, tab + a.f.twoff[0]);
    // zeros: nh .. n - nh, and the padding n .. N - 1
    const int nz = n - 2 * nh + 1, nzt = nz + N - n;
    for (int idx = threadIdx.x; idx < TB * nzt; idx += NT) {
        const int tr = idx / nzt, z = idx - tr * nzt;
        X[tr * N + (z < nz ? nh + z : n + z - nz)] = mk<T>(T(0), T(0));
    }
#pragma unroll
    for (int t = 0; t < PL; ++t) {
        const int idx = threadIdx.x + t * NT;
        const int tr = idx / NHC, k = idx % NHC;
        if (idx >= TB * NHC || k >= nh) continue;
        V *xr = X + tr * N;
        if (k == 0) {
            xr[0] = mk<T>(x1[t], x2[t]);  // c_0 = 1
        } else {
            xr[k] = cmul(mk<T>(x1[t] - y2[t], y1[t] + x2[t]), chirp[k]);
            xr[n - k] = cmul(mk<T>(x1[t] + y2[t], x2[t] - y1[t]), chirp[n - k]);
        }
    }
    __syncthreads();
    __builtin_amdgcn_s_setprio(0);
    blue_conv<T, FI, TB, NT, true, 0, 1>(X, tw, H, T(1));
    {
        // transposed stage 0 of the inverse, the products, stage 0 of the forward
        const T a0 = T(a.A0[0]);
        const T da = T(a.D[0]);
        const auto *g = gbl(reinterpret_cast<const T *>(a.g) + (long)2 * pr0 * n);
        for (int idx = threadIdx.x; idx < TQ * TB; idx += NT) {
            const int tr = idx / TQ, i = idx % TQ;
            const int p = tr % PW;
            const bool v1 = 2 * p < nrow_wg, v2 = 2 * p + 1 < nrow_wg;
            V *xr = X + tr * N + i * R;
            T g1[R], g2[R];
#pragma unroll
            for (int q = 0; q < R; ++q) {  // points past the row and missing rows read entry 0
                const int x = i + q * TQ;
                g1[q] = g[x < n && v1 ? 2 * p * n + x : 0];
                g2[q] = g[x < n && v2 ? (2 * p + 1) * n + x : 0];
            }
            V u[R];
#pragma unroll
            for (int q = 0; q < R; ++q) u[q] = xr[q];
            dftn<T, R>(u, T(1));
#pragma unroll
            for (int q = 0; q < R; ++q) {
                const int x = i + q * TQ;
                const V c = chirp[x < n ? x : 0];
                V v = cmul(u[q], c);
                v.x *= a0 + g1[q] * da;
                v.y *= a0 + g2[q] * da;
                v = cmul(v, mk<T>(c.x, -c.y));
                u[q] = x < n ? v : mk<T>(T(0), T(0));
            }
            dftn<T, R>(u, T(-1));
#pragma unroll
            for (int q = 0; q < R; ++q) xr[q] = u[q];
        }
        __syncthreads();
    }
    blue_conv<T, FI, TB, NT, true, 1, 0>(X, tw, H, T(-1));
    const T half = T(a.scale) * T(0.5);
    for (int idx = threadIdx.x; idx < TB * NHC; idx += NT) {
        const int tr = idx / NHC, k = idx % NHC;
        const int c = tr / PW, p = tr % PW;
        if (k >= nh || 2 * p >= nrow_wg) continue;
        const int km = k == 0 ? 0 : n - k;
        const V w = cmul(X[tr * N + k], chirp_at<T>(chirp, k, T(-1)));
        const V wm = cmul(X[tr * N + km], chirp_at<T>(chirp, km, T(-1)));
        auto *o = data + (long)c * a.cs + 2 * p * nh + k;
        gst(o, mk<T>((w.x + wm.x) * half, (w.y - wm.y) * half));
        if (2 * p + 1 < nrow_wg) gst(o + nh, mk<T>((w.y + wm.y) * half, (wm.x - w.x) * half));
    }
}

// ---- launchers and the table of a part ----
template <typename T, int FI, int D, bool BLUE, bool TWO = false>
void launch_pencil_t(const PencilArgs *args, const int *woff, int np, int total, hipStream_t s, LaunchEv ev) {
    constexpr int N = kFastSched[FI].n, G = TWO ? 1 : D;
    dispatch((pencil_fast<T, FI, D, BLUE, TWO>), dim3(total), dim3(pencil_nt(N, sizeof(Vt<T>), G, BLUE)),
             pencil_lds(N, sizeof(Vt<T>), G, BLUE), Disp(s, ev), args, woff, np);
}

template <typename T, int FI, int D>
void launch_blue_row_t(const RowArgs *args, const int *woff, int np, int total, hipStream_t s, LaunchEv ev) {
    dispatch((row_iso_blue<T, FI, D>), dim3(total), dim3(blue_nt(FI, sizeof(Vt<T>), D)), blue_lds(FI, sizeof(Vt<T>), D),
             Disp(s, ev), args, woff, np);
}

template <typename T, int FI, int D>
void launch_row_t(const RowArgs *args, const int *woff, int np, int total, hipStream_t s, LaunchEv ev) {
    dispatch((row_fast<T, FI, D>), dim3(total), dim3(kThreads), row_lds(kFastSched[FI].n, sizeof(Vt<T>), D),
             Disp(s, ev), args, woff, np);
}

template <typename T, int FI>
void launch_iso_t(const RowArgs *args, const int *woff, int np, int total, hipStream_t s, LaunchEv ev) {
    if constexpr (kFastSched[FI].nst == 2)
        dispatch((row_iso_split<T, FI>), dim3(total), dim3(split_nt(FI)), iso_lds<T>(FI), Disp(s, ev), args, woff, np);
    else
        dispatch((row_iso_fast<T, FI>), dim3(total), dim3(iso_nt(FI)), iso_lds<T>(FI), Disp(s, ev), args, woff, np);
}

template <typename T, int FI, int D>
void launch_staged_t(const RowArgs *args, const int *woff, int np, int total, hipStream_t s, LaunchEv ev) {
    dispatch((row_iso_staged<T, FI, D>), dim3(total), dim3(staged_nt(FI, D, sizeof(Vt<T>))), staged_lds<T>(FI, D),
             Disp(s, ev), args, woff, np);
}

template <typename T, int FI, int D>
void launch_pairs_t(const RowArgs *args, const int *woff, int np, int total, hipStream_t s, LaunchEv ev) {
    dispatch((row_iso_pairs<T, FI, D>), dim3(total), dim3(pairs_nt(FI, sizeof(Vt<T>), D)),
             pairs_lds(FI, sizeof(Vt<T>), D), Disp(s, ev), args, woff, np);
}

template <typename T, int FI>
void launch_plane_t(const RowArgs *args, const int *woff, int np, int total, hipStream_t s, LaunchEv ev) {
    constexpr int N = kFastSched[FI].n;
    dispatch((plane_iso<T, FI>), dim3(total), dim3(plane_nt(N)), plane_lds(N, sizeof(Vt<T>)), Disp(s, ev), args, woff, np);
}

template <int FI, int D>
void launch_gram_t(const RowArgs *args, const int *woff, int np, int total, hipStream_t s, LaunchEv ev) {
    dispatch((row_gram_fast<double, FI, D>), dim3(total), dim3(kThreads), gram_lds(kFastSched[FI].n, D), Disp(s, ev),
             args, woff, np);
}

template <typename T, int FI, int D>
void fill_dim(FastKernels &k) {
    constexpr int n = kFastSched[FI].n, es = sizeof(Vt<T>), p = sizeof(T) == 8;
    if constexpr (fast_dim(FI, D)) {
        k.pencil[p][D - 2] = {launch_pencil_t<T, FI, D, false>, pencil_batch(n, es, D), pencil_lds(n, es, D)};
        if constexpr (D == 3)
            k.pencil2[p] = {launch_pencil_t<T, FI, D, false, true>, pencil_batch(n, es, 1), pencil_lds(n, es, 1)};
        if constexpr (D == 3 && has_blue(FI, D))
            k.blue_pencil2[p] = {launch_pencil_t<T, FI, D, true, true>, pencil_batch(n, es, 1, true),
                                 pencil_lds(n, es, 1, true)};
        if constexpr (has_blue(FI, D)) {
            k.blue_pencil[p][D - 2] = {launch_pencil_t<T, FI, D, true>, pencil_batch(n, es, D, true),
                                       pencil_lds(n, es, D, true)};
            k.blue_row[p][D - 2] = {launch_blue_row_t<T, FI, D>, blue_tb(n, es, D), ((n + 1) / 2 + 1) / 2,
                                    blue_lds(FI, es, D)};
        }
        k.row[p][D - 2] = {launch_row_t<T, FI, D>, fast_batch(n, es, D), (n + 1) / 2, row_lds(n, es, D)};
        if constexpr (has_staged(FI))
            k.pairs[p][D - 2] = {launch_staged_t<T, FI, D>, staged_tb(FI, D, es), staged_nhc(n), staged_lds<T>(FI, D)};
        else if constexpr (has_pairs(FI))
            (pairs_one(n, es, D) ? k.iso : k.pairs)[p][D - 2] = {launch_pairs_t<T, FI, D>, pairs_tb(n, es, D),
                                                                 (n + 1) / 2, pairs_lds(FI, es, D)};
        if constexpr (D == 3 && has_plane(n))
            k.plane[p] = {launch_plane_t<T, FI>, 1, staged_nhc(n), plane_lds(n, es)};
        if constexpr (has_iso(FI)) k.iso[p][D - 2] = {launch_iso_t<T, FI>, iso_tb(FI), (n + 1) / 2, iso_lds<T>(FI)};
    }
}

template <int FI>
void fill_length(FastKernels &k) {
    constexpr int n = kFastSched[FI].n;
    fill_dim<double, FI, 2>(k);
    fill_dim<double, FI, 3>(k);
    fill_dim<float, FI, 2>(k);
    fill_dim<float, FI, 3>(k);
    k.gram[0] = {launch_gram_t<FI, 2>, gram_batch(n, 16, 2), (n + 1) / 2, gram_lds(n, 2)};
    if constexpr (fast_dim(FI, 3)) k.gram[1] = {launch_gram_t<FI, 3>, gram_batch(n, 16, 3), (n + 1) / 2, gram_lds(n, 3)};
}

template <int FI>
void fill_from(FastKernels *t) {
    if constexpr (FI < kNumFast) {
        fill_length<FI>(t[FI]);
        fill_from<FI + kFastParts>(t);
    }
}

}  // namespace

template <> void fill_fast<FFTGAL_PART>(FastKernels *table) { fill_from<FFTGAL_PART>(table); }

}  // namespace fftgal
