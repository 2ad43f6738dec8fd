// HIP kernels for gfx950: the double-grid Ga operator (Algorithm 2) as
// fused FFT passes, conjugate-gradient vector kernels, FP64 energy quadrature,
// and the material setup (eq. MBA_GA, eq. inclcomp_formula, Lemma grid_compos).
//
// Transforms are mixed-radix (3, 5, 7) self-sorting Stockham DFTs staged in
// LDS; every grid size is odd (M >= 2N-1 odd and 3,5,7-smooth), so no radix 2
// and no Nyquist frequency ever occurs.
#include "fftgal_device.h"

#include <utility>

#include <algorithm>
#include <cmath>

namespace fftgal {
namespace {
// One Stockham stage of radix R over nb independent transforms of length n.
// Butterfly i (k = i mod p) reads positions i + q n/R, applies the twiddles
// exp(sg 2 pi i q k / (p R)), a length-R DFT, and writes positions
// (i - k) R + k + q p.  ROWL: element (pos, b) at b*n + pos, else pos*nb + b.
template <typename T, int R, bool ROWL>
__device__ __forceinline__ void stage(const Vt<T> *X, Vt<T> *Y, int n, int p, int nb,
                                      const Vt<T> *__restrict__ tw, T sg) {
    const int Tq = n / R;
    const int total = Tq * nb;
    for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
        int i, b;
        if (ROWL) {
            b = idx / Tq;
            i = idx - b * Tq;
        } else {
            i = idx / nb;
            b = idx - i * nb;
        }
        const int k = i % p;
        Vt<T> u[R];
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int pos = i + q * Tq;
            u[q] = ROWL ? X[b * n + pos] : X[pos * nb + b];
        }
        if (p > 1) {
#pragma unroll
            for (int q = 1; q < R; ++q) {
                Vt<T> w = tw[(q - 1) * p + k];
                w.y *= -sg;  // table holds exp(-2 pi i q k / (p R))
                u[q] = cmul(u[q], w);
            }
        }
        dftn<T, R>(u, sg);
        const int j = (i - k) * R + k;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int pos = j + q * p;
            if (ROWL)
                Y[b * n + pos] = u[q];
            else
                Y[pos * nb + b] = u[q];
        }
    }
}

// The stages of a transform of length f.L in LDS, ping-ponging between A and
// Bf; returns the buffer holding the result.  P13: lengths with the factors 11 or
// 13 too; lengths that have them do not use radix 25.
template <typename T, bool ROWL, bool P13>
__device__ __forceinline__ Vt<T> *fft_stages(Vt<T> *A, Vt<T> *Bf, const FftDesc &f, int nb, const Vt<T> *tw, T sg,
                                              int tb = 0) {
    Vt<T> *X = A;
    Vt<T> *Y = Bf;
    int p = 1;
    for (int s = 0; s < f.nst; ++s) {
        const int r = f.radix[s];
        const Vt<T> *t = tw + (f.twoff[s] - tb);
        switch (r) {
            case 3: stage<T, 3, ROWL>(X, Y, f.L, p, nb, t, sg); break;
            case 5: stage<T, 5, ROWL>(X, Y, f.L, p, nb, t, sg); break;
            case 7: stage<T, 7, ROWL>(X, Y, f.L, p, nb, t, sg); break;
            case 9: stage<T, 9, ROWL>(X, Y, f.L, p, nb, t, sg); break;
            case 15: stage<T, 15, ROWL>(X, Y, f.L, p, nb, t, sg); break;
            default:
                if constexpr (P13) {
                    if (r == 11)
                        stage<T, 11, ROWL>(X, Y, f.L, p, nb, t, sg);
                    else
                        stage<T, 13, ROWL>(X, Y, f.L, p, nb, t, sg);
                } else {
                    stage<T, 25, ROWL>(X, Y, f.L, p, nb, t, sg);
                }
        }
        __syncthreads();
        Vt<T> *tmp = X;
        X = Y;
        Y = tmp;
        p *= r;
    }
    return X;
}

// Full transform of nb sequences of length f.n in LDS (positions 0 .. n - 1 of
// buffers of f.L positions; ROWL: element (pos, b) at b L + pos, else
// pos nb + b); returns the buffer holding the result.  Must be called by
// every thread of the work-group.
template <typename T, bool ROWL, bool P13>
__device__ __forceinline__ Vt<T> *fft_lds(Vt<T> *A, Vt<T> *Bf, const FftDesc &f, int nb, const Vt<T> *tw, T sg,
                                           int tb = 0) {
    if (P13 || !f.blue) return fft_stages<T, ROWL, P13>(A, Bf, f, nb, tw, sg, tb);
    // Bluestein: u_j = x_j c_j zero-padded to L, H (.) DFT^- u, DFT^+, times c_k
    const int n = f.n, L = f.L;
    const Vt<T> *chirp = tw + (f.choff - tb);
    const Vt<T> *H = tw + (f.hoff - tb);
    auto at = [&](Vt<T> *buf, int pos, int b) -> Vt<T> & { return ROWL ? buf[b * L + pos] : buf[pos * nb + b]; };
    auto chirp_of = [&](int m) {  // c_m for the sign sg
        Vt<T> c = chirp[m];
        c.y *= sg;
        return c;
    };
    for (int idx = threadIdx.x; idx < L * nb; idx += blockDim.x) {
        const int b = idx / L, pos = idx - b * L;
        Vt<T> &v = at(A, pos, b);
        v = pos < n ? cmul(v, chirp_of(pos)) : mk<T>(T(0), T(0));
    }
    __syncthreads();
    Vt<T> *X = fft_stages<T, ROWL, false>(A, Bf, f, nb, tw, T(-1), tb);
    for (int idx = threadIdx.x; idx < L * nb; idx += blockDim.x) {
        const int b = idx / L, k = idx - b * L;
        // H for the sign sg: H_k (sg = +1) or conj(H_{-k}) (sg = -1)
        Vt<T> h = H[sg > T(0) ? k : (k == 0 ? 0 : L - k)];
        if (sg < T(0)) h.y = -h.y;
        Vt<T> &v = at(X, k, b);
        v = cmul(v, h);
    }
    __syncthreads();
    Vt<T> *Y = fft_stages<T, ROWL, false>(X, X == A ? Bf : A, f, nb, tw, T(1), tb);
    for (int idx = threadIdx.x; idx < n * nb; idx += blockDim.x) {
        const int b = idx / n, pos = idx - b * n;
        Vt<T> &v = at(Y, pos, b);
        v = cmul(v, chirp_of(pos));
    }
    __syncthreads();
    return Y;
}

// ---------------------------------------------------------------------------
// Pencil pass: batched DFT along a strided axis.
// ---------------------------------------------------------------------------
// t[al] for a runtime component al < 3 without indexing a private array
template <typename T>
__device__ __forceinline__ T pick3(const T *t, int al) {
    return al == 0 ? t[0] : (al == 1 ? t[1] : t[2]);
}

// two waves per SIMD: the radix-25 stage alone would take the register
// file of one.  The components of a pencil are transformed a.cb at a time in
// one batch of cb * B sequences (layout: position * (cn B) + j B + b for
// component al0 + j of the chunk), so that a small grid runs one chain of
// stages and barriers per work-group instead of one per component.
template <typename T, bool P13>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void pencil_kernel(PencilArgs a) {
    using V = Vt<T>;
    if (a.status != nullptr && a.status->done) return;
    extern __shared__ __align__(16) unsigned char smem_raw[];  // 16-byte complex doubles
    const int n = a.f.n;
    const int B = a.B;
    const int cb = a.cb;
    V *bufA = reinterpret_cast<V *>(smem_raw);
    V *bufB = bufA + (size_t)a.f.L * cb * B;
    V *acc = bufB + (size_t)a.f.L * cb * B;
    const int b0 = blockIdx.x * B;
    const int o = blockIdx.y;
    const int nbw = min(B, a.nb - b0);
    const V *tw = reinterpret_cast<const V *>(a.tw);
    // the transform's table entries (stage twiddles; Bluestein chirp and
    // filter) staged in LDS after the buffers when they fit (a.twl entries from
    // entry twoff[0]); visible to the stages after the loads' barrier
    int tb = 0;
    if (a.twl > 0) {
        int lacc = 0;
        if (a.pro == PRO_EXPAND) lacc = a.nc * a.L_in;
        if (a.epi == EPI_PROJECT) lacc = a.nc * a.L_out;
        V *twl = acc + (size_t)lacc * B;
        tb = a.f.twoff[0];
        for (int i = threadIdx.x; i < a.twl; i += blockDim.x) twl[i] = tw[tb + i];
        tw = twl;
    }
    const T sg = T(a.sgn);
    const T scale = T(a.scale);
    const V *in = reinterpret_cast<const V *>(a.in);
    V *out = reinterpret_cast<V *>(a.out);
    const V zero = mk<T>(T(0), T(0));

    auto freq = [&](int l, int L, int b, int *k1, int *k2, int *k3) {
        *k1 = wrapi(l, L);
        if (a.d == 3) {
            *k2 = wrapi(b / a.Nh, a.Nmid);
            *k3 = b % a.Nh;
        } else {
            *k2 = b % a.Nh;
            *k3 = 0;
        }
    };

    if (a.pro == PRO_EXPAND) {
        // c_a -> e_alpha = i sum_a t_a(k)_alpha c_a on Z_N, zero-padded to n.
        const V *sr = reinterpret_cast<const V *>(a.st_r);
        V *sp = reinterpret_cast<V *>(a.st_p);
        const V *sx = reinterpret_cast<const V *>(a.st_x);
        const T beta = (a.update_p && a.status) ? T(a.status->beta) : T(0);
        for (int s = 0; s < a.nsol; ++s) {
            for (int idx = threadIdx.x; idx < a.nc * a.L_in * B; idx += blockDim.x) {
                const int bb = idx % B;
                const int l = (idx / B) % a.L_in;
                const int c = idx / (B * a.L_in);
                V v = zero;
                if (bb < nbw) {
                    const long off = s * a.st_ss + c * a.st_cs + (long)l * a.in_ls + b0 + bb;
                    if (a.update_p) {
                        const V r = sr[off];
                        const V pv = sp[off];
                        v = mk<T>(r.x + beta * pv.x, r.y + beta * pv.y);
                        sp[off] = v;
                    } else {
                        v = sx[off];
                    }
                }
                acc[(c * a.L_in + l) * B + bb] = v;
            }
            __syncthreads();
            for (int al0 = 0; al0 < a.ncomp; al0 += cb) {
                const int cn = min(cb, a.ncomp - al0);
                const int nbt = cn * B;
                for (int idx = threadIdx.x; idx < n * nbt; idx += blockDim.x) bufA[idx] = zero;
                __syncthreads();
                for (int idx = threadIdx.x; idx < a.L_in * B; idx += blockDim.x) {
                    const int bb = idx % B;
                    const int l = idx / B;
                    if (bb >= nbw) continue;
                    int k1, k2, k3;
                    freq(l, a.L_in, b0 + bb, &k1, &k2, &k3);
                    T t[2][3];
                    const int nt = basis<T>(a.d, a.kind, k1, k2, k3, t);
                    double pc = 1.0, ps = 0.0;
                    if (has_shift(a)) shift_phase(a, k1, k2, k3, &pc, &ps);
                    V *dst = bufA + posmod(k1, n) * nbt + bb;
                    for (int j = 0; j < cn; ++j) {
                        const int al = al0 + j;
                        T ex = T(0), ey = T(0);
#pragma unroll
                        for (int c = 0; c < 2; ++c) {
                            if (c >= nt) break;
                            const V cv = acc[(c * a.L_in + l) * B + bb];
                            const T tc = pick3<T>(t[c], al);
                            ex -= tc * cv.y;  // i * t * c
                            ey += tc * cv.x;
                        }
                        if (has_shift(a)) {
                            const T nx = ex * T(pc) - ey * T(ps);
                            ey = ex * T(ps) + ey * T(pc);
                            ex = nx;
                        }
                        dst[j * B] = mk<T>(ex, ey);
                    }
                }
                __syncthreads();
                V *res = fft_lds<T, false, P13>(bufA, bufB, a.f, nbt, tw, sg, tb);
                for (int idx = threadIdx.x; idx < a.L_out * nbt; idx += blockDim.x) {
                    const int bt = idx % nbt;
                    const int l = idx / nbt;
                    const int j = cn > 1 ? bt / B : 0;  // no division for one component
                    const int bb = bt - j * B;
                    if (bb >= nbw) continue;
                    const int pos = posmod(wrapi(l, a.L_out), n);
                    V v = res[pos * nbt + bt];
                    v.x *= scale;
                    v.y *= scale;
                    const long cbase = (long)(s * a.ncomp + al0 + j) * a.out_cs + (long)o * a.out_os + b0;
                    out[cbase + (long)l * a.out_ls + bb] = v;
                }
                __syncthreads();
            }
        }
        return;
    }

    // PRO_PLAIN
    if (a.epi == EPI_PROJECT) {
        for (int idx = threadIdx.x; idx < a.nc * a.L_out * B; idx += blockDim.x) acc[idx] = zero;
    }
    double part = 0.0;
    for (int al0 = 0; al0 < a.ncomp; al0 += cb) {
        const int cn = min(cb, a.ncomp - al0);
        const int nbt = cn * B;
        if (a.L_in < n) {
            for (int idx = threadIdx.x; idx < n * nbt; idx += blockDim.x) bufA[idx] = zero;
            __syncthreads();
        }
        for (int idx = threadIdx.x; idx < a.L_in * nbt; idx += blockDim.x) {
            const int bt = idx % nbt;
            const int l = idx / nbt;
            const int j = cn > 1 ? bt / B : 0;
            const int bb = bt - j * B;
            V v = zero;
            if (bb < nbw) v = in[(long)(al0 + j) * a.in_cs + (long)o * a.in_os + b0 + (long)l * a.in_ls + bb];
            bufA[posmod(wrapi(l, a.L_in), n) * nbt + bt] = v;
        }
        __syncthreads();
        V *res = fft_lds<T, false, P13>(bufA, bufB, a.f, nbt, tw, sg, tb);
        if (a.epi == EPI_PROJECT) {
            // q_a += -i t_a(k)_alpha yhat_alpha(k) on Z_N, alpha in ascending order
            for (int idx = threadIdx.x; idx < a.L_out * B; idx += blockDim.x) {
                const int bb = idx % B;
                const int l = idx / B;
                if (bb >= nbw) continue;
                int k1, k2, k3;
                freq(l, a.L_out, b0 + bb, &k1, &k2, &k3);
                T t[2][3];
                const int nt = basis<T>(a.d, a.kind, k1, k2, k3, t);
                const V *src = res + posmod(k1, n) * nbt + bb;
                for (int j = 0; j < cn; ++j) {
                    const V y = src[j * B];
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        if (c >= nt) break;
                        V &q = acc[(c * a.L_out + l) * B + bb];
                        const T tt = pick3<T>(t[c], al0 + j) * scale;
                        q.x += tt * y.y;
                        q.y -= tt * y.x;
                    }
                }
            }
        } else {
            for (int idx = threadIdx.x; idx < a.L_out * nbt; idx += blockDim.x) {
                const int bt = idx % nbt;
                const int l = idx / nbt;
                const int j = cn > 1 ? bt / B : 0;
                const int bb = bt - j * B;
                if (bb >= nbw) continue;
                const int kk = wrapi(l, a.L_out);
                V v = res[posmod(kk, n) * nbt + bt];
                T sc = scale;
                if (a.epi == EPI_WINDOW) {
                    int k1, k2, k3;
                    freq(l, a.L_out, b0 + bb, &k1, &k2, &k3);
                    double w = a.winscale * sinc_pi((double)k1 / a.Pw[0]) * sinc_pi((double)k2 / a.Pw[1]);
                    if (a.d == 3) w *= sinc_pi((double)k3 / a.Pw[2]);
                    sc = T(w * a.scale);
                }
                v.x *= sc;
                v.y *= sc;
                const long obase = (long)(al0 + j) * a.out_cs + (long)o * a.out_os + b0;
                out[obase + (long)l * a.out_ls + bb] = v;
            }
        }
        __syncthreads();
    }
    if (a.epi == EPI_PROJECT) {
        V *q = out;
        const V *dv = reinterpret_cast<const V *>(a.st_dot);
        for (int idx = threadIdx.x; idx < a.nc * a.L_out * B; idx += blockDim.x) {
            const int bb = idx % B;
            const int l = (idx / B) % a.L_out;
            const int c = idx / (B * a.L_out);
            if (bb >= nbw) continue;
            V v = acc[idx];
            const long off = (long)c * a.out_cs + (long)l * a.out_ls + b0 + bb;
            if (has_shift(a)) {  // S*(s): the conjugate phase
                int k1, k2, k3;
                freq(l, a.L_out, b0 + bb, &k1, &k2, &k3);
                double pc, ps;
                shift_phase(a, k1, k2, k3, &pc, &ps);
                const T nx = v.x * T(pc) + v.y * T(ps);
                v.y = v.y * T(pc) - v.x * T(ps);
                v.x = nx;
            }
            if (a.accumulate) {
                const V old = q[off];
                v.x += old.x;
                v.y += old.y;
            }
            q[off] = v;
            const int klast = (b0 + bb) % a.Nh;
            const double w = klast == 0 ? 1.0 : 2.0;
            if (dv != nullptr) {
                const V pv = dv[off];
                part += w * ((double)pv.x * (double)v.x + (double)pv.y * (double)v.y);
            } else {
                part += w * ((double)v.x * (double)v.x + (double)v.y * (double)v.y);
            }
        }
        const double s = block_sum(part);
        if (threadIdx.x == 0) a.partial[blockIdx.y * gridDim.x + blockIdx.x] = s;
    }
}

// Voxel value as seen by the material series: the conductivity itself (0), the
// indicator of the high phase of a two-phase image (1), the inverse
// conductivity (2), or zero (3, a one-phase image).
template <typename T>
__device__ __forceinline__ T map_voxel(T v, int mode, double vmax) {
    if (mode == 1) return v == T(vmax) ? T(1) : T(0);
    if (mode == 2) return T(1) / v;
    if (mode == 3) return T(0);
    return v;
}

// GaNi material (Def. GaNi: the rectangle rule samples A at the grid points).
__global__ __launch_bounds__(kThreads) void sample_incl_kernel(double *g, int d, int m0, int m1, int m2,
                                                               const InclDev *inc, int n, double w0) {
    const long total = (long)m0 * m1 * m2;
    for (long idx = blockIdx.x * (long)kThreads + threadIdx.x; idx < total; idx += (long)gridDim.x * kThreads) {
        const int j2 = (int)(idx % m2);
        const int j1 = (int)((idx / m2) % m1);
        const int j0 = (int)(idx / ((long)m2 * m1));
        double x[3];
        x[0] = (double)wrapi(j0, m0) / m0;
        x[1] = (double)wrapi(j1, m1) / m1;
        x[2] = (double)wrapi(j2, m2) / m2;  // 2D: m2 = 1, x[2] unused
        double v = w0;
        for (int i = 0; i < n; ++i) {
            double r2 = 0.0;
            bool inside = true;
            for (int a = 0; a < d; ++a) {
                double dx = x[a] - inc[i].c[a];
                dx -= rint(dx);
                if (inc[i].shape == 0)
                    inside = inside && fabs(dx) < 0.5 * inc[i].h[a];
                else
                    r2 += dx * dx;
            }
            if (inc[i].shape != 0) inside = r2 < inc[i].h[0] * inc[i].h[0];
            if (inside) v += inc[i].w;
        }
        g[idx] = v;
    }
}

__global__ __launch_bounds__(kThreads) void sample_voxel_kernel(double *g, const double *img, int p0, int p1, int p2,
                                                                int m0, int m1, int m2, int map, double vmax) {
    const long total = (long)m0 * m1 * m2;
    for (long idx = blockIdx.x * (long)kThreads + threadIdx.x; idx < total; idx += (long)gridDim.x * kThreads) {
        const int j2 = (int)(idx % m2);
        const int j1 = (int)((idx / m2) % m1);
        const int j0 = (int)(idx / ((long)m2 * m1));
        const int q0 = posmod((int)rint((double)wrapi(j0, m0) * p0 / m0), p0);
        const int q1 = posmod((int)rint((double)wrapi(j1, m1) * p1 / m1), p1);
        const int q2 = posmod((int)rint((double)wrapi(j2, m2) * p2 / m2), p2);
        g[idx] = map_voxel<double>(img[((long)q0 * p1 + q1) * p2 + q2], map, vmax);
    }
}

// Upper and lower voxel images (Remark adjusting_A).
__global__ __launch_bounds__(kThreads) void envelope_kernel(double *up, double *lo, int d, int p0, int p1, int p2,
                                                            const InclDev *inc, int n, const double *ext) {
    const long total = (long)p0 * p1 * p2;
    for (long idx = blockIdx.x * (long)kThreads + threadIdx.x; idx < total; idx += (long)gridDim.x * kThreads) {
        const int j2 = (int)(idx % p2);
        const int j1 = (int)((idx / p2) % p1);
        const int j0 = (int)(idx / ((long)p2 * p1));
        const int pp[3] = {p0, p1, p2};
        const double x[3] = {(double)wrapi(j0, p0) / p0, (double)wrapi(j1, p1) / p1, (double)wrapi(j2, p2) / p2};
        double hi = -HUGE_VAL, lw = HUGE_VAL;
        bool matrix = true;
        for (int i = 0; i < n; ++i) {
            bool meets = true, contains = true;
            double near2 = 0.0, far2 = 0.0;
            for (int a = 0; a < d; ++a) {
                double dc = x[a] - inc[i].c[a];
                dc = fabs(dc - rint(dc));
                const double half = 0.5 / pp[a];
                if (inc[i].shape == 0) {
                    meets = meets && dc < 0.5 * inc[i].h[a] + half;
                    contains = contains && dc + half <= 0.5 * inc[i].h[a];
                } else {
                    // unfused, so that a voxel exactly on the circle is classified
                    // as in plain rounded arithmetic
                    const double nr = fmax(dc - half, 0.0), fr = dc + half;
                    near2 = __dadd_rn(near2, __dmul_rn(nr, nr));
                    far2 = __dadd_rn(far2, __dmul_rn(fr, fr));
                }
            }
            if (inc[i].shape != 0) {
                const double r2 = __dmul_rn(inc[i].h[0], inc[i].h[0]);
                meets = near2 < r2;
                contains = far2 <= r2;
            }
            if (meets) {
                hi = fmax(hi, ext[2 + 2 * i]);
                lw = fmin(lw, ext[3 + 2 * i]);
            }
            if (contains) matrix = false;
        }
        if (matrix) {
            hi = fmax(hi, ext[0]);
            lw = fmin(lw, ext[1]);
        }
        up[idx] = hi;
        lo[idx] = lw;
    }
}

// Reduced Ga material: fold the series on Z_{2N-1} onto Z_N with the phase of
// shift s (one output frequency per thread; at most two sources per axis).
// Index 2 is always the last axis; index 1 is used in 3D only.
__global__ __launch_bounds__(kThreads) void fold_series_kernel(double2 *out, const double2 *coef, int d, int n0,
                                                               int n1, int n2, int l0, int l1, int lh, int s0, int s1,
                                                               int s2) {
    const int nh = (n2 + 1) / 2;  // stored output entries along the last axis
    const long total = (d == 3 ? (long)n0 * n1 : (long)n0) * nh;
    const int nn[3] = {n0, n1, n2};
    const int sh[3] = {s0, d == 3 ? s1 : 0, s2};
    for (long idx = blockIdx.x * (long)kThreads + threadIdx.x; idx < total; idx += (long)gridDim.x * kThreads) {
        const int m2 = (int)(idx % nh);
        const long r = idx / nh;
        const int m1 = d == 3 ? (int)(r % n1) : 0;
        const int m0 = d == 3 ? (int)(r / n1) : (int)r;
        const int jj[3] = {wrapi(m0, n0), d == 3 ? wrapi(m1, n1) : 0, m2};
        // sources k_a = j_a and j_a -/+ N_a (for j_a != 0): |k_a| <= N_a - 1
        int ka[3][2], na[3];
        for (int a = 0; a < 3; ++a) {
            ka[a][0] = jj[a];
            ka[a][1] = jj[a] > 0 ? jj[a] - nn[a] : jj[a] + nn[a];
            na[a] = (jj[a] != 0 && (a != 1 || d == 3)) ? 2 : 1;
        }
        double re = 0.0, im = 0.0;
        for (int i0 = 0; i0 < na[0]; ++i0)
            for (int i1 = 0; i1 < na[1]; ++i1)
                for (int i2 = 0; i2 < na[2]; ++i2) {
                    const int k0 = ka[0][i0], k1 = ka[1][i1], k2 = ka[2][i2];
                    // stored entries have k_last >= 0; the others by conjugate symmetry
                    const bool cj = k2 < 0;
                    const int q0 = cj ? -k0 : k0, q1 = cj ? -k1 : k1, q2 = cj ? -k2 : k2;
                    double2 v = d == 3 ? coef[((long)posmod(q0, l0) * l1 + posmod(q1, l1)) * lh + q2]
                                       : coef[(long)posmod(q0, l0) * lh + q2];
                    if (cj) v.y = -v.y;
                    const double x = (sh[0] ? (double)k0 / nn[0] : 0.0) + (sh[1] ? (double)k1 / nn[1] : 0.0) +
                                     (sh[2] ? (double)k2 / nn[2] : 0.0);
                    double ps, pc;
                    sincospi(-x, &ps, &pc);
                    re += v.x * pc - v.y * ps;
                    im += v.x * ps + v.y * pc;
                }
        out[idx] = make_double2(re, im);
    }
}

// ---------------------------------------------------------------------------
// Row pass: real transforms along the last axis, two rows per complex DFT.
// ---------------------------------------------------------------------------
// Transform buffers (components) of the generic row kernel.
__host__ __device__ inline int row_zbufs(const RowArgs &a) {
    if (a.mode == ROW_RHS) return a.d;
    if (a.mode == ROW_R2C || a.mode == ROW_C2R) return 1;
    if (a.mode == ROW_GRAM && a.gpack) return (a.ncomp + 1) / 2;
    return a.ncomp;
}

template <typename T, int DIM, bool P13>
__global__ __launch_bounds__(kThreads) void row_kernel(RowArgs a) {
    using V = Vt<T>;
    if (a.status != nullptr && a.status->done) return;
    extern __shared__ __align__(16) unsigned char smem_raw[];  // 16-byte complex doubles
    const int n = a.f.n;
    const int ln = a.f.L;  // buffer length per transform (n unless Bluestein)
    const int RP = a.RP;
    const int nh = a.Nh_row;
    // one buffer per component (Z[c] = Z + c RP ln) and the transforms'
    // scratch S: RP ln (a batch per component) or the size of Z (zbatch: the
    // rows of all components form one batch, sequence c RP + j at (c RP + j) ln)
    const bool zb = a.zbatch != 0;
    const int nzb = row_zbufs(a);
    V *const S = reinterpret_cast<V *>(smem_raw) + (zb ? (size_t)nzb * RP * ln : 0);
    V *const Z = reinterpret_cast<V *>(smem_raw) + (zb ? 0 : (size_t)RP * ln);
    const V *tw = reinterpret_cast<const V *>(a.tw);
    V *data = reinterpret_cast<V *>(a.data);
    const T *g = reinterpret_cast<const T *>(a.g);
    const int pair0 = blockIdx.x * RP;
    const int npairs_total = (a.nrows + 1) / 2;
    const int nvp = min(RP, npairs_total - pair0);
    const V zero = mk<T>(T(0), T(0));
    constexpr int d = DIM;  // the material and field loops unroll (no private arrays)
    const int nzc = (a.mode == ROW_RHS || a.mode == ROW_R2C) ? (a.mode == ROW_RHS ? d : 1) : a.ncomp;

    auto zbuf = [&](int c) { return Z + (size_t)c * RP * ln; };
    auto fft_into = [&](int c, T sg) {
        V *res = fft_lds<T, true, P13>(zbuf(c), S, a.f, RP, tw, sg);
        if (res != zbuf(c)) {
            for (int idx = threadIdx.x; idx < RP * ln; idx += blockDim.x) zbuf(c)[idx] = res[idx];
            __syncthreads();
        }
    };

    if (a.mode == ROW_GRAM && a.gpack) {
        // (A_M (E_s + e_s), E_t + e_t) with components 2 c2 and 2 c2 + 1 of one
        // row packed per transform (z = u_{2 c2} + i u_{2 c2 + 1}); row r0 + j
        const int r0 = blockIdx.x * RP;
        const int nvr = min(RP, a.nrows - r0);
        const int npk = (a.ncomp + 1) / 2;
        for (int c2 = 0; c2 < npk; ++c2) {
            V *zc = zbuf(c2);
            for (int idx = threadIdx.x; idx < RP * ln; idx += blockDim.x) zc[idx] = zero;
            __syncthreads();
            const bool two = 2 * c2 + 1 < a.ncomp;
            for (int idx = threadIdx.x; idx < RP * nh; idx += blockDim.x) {
                const int j = idx / nh;
                const int kx = idx - j * nh;
                if (j >= nvr) continue;
                const long row = (long)(r0 + j) * nh + kx;
                const V u1 = data[(long)(2 * c2) * a.cs + row];
                const V u2 = two ? data[(long)(2 * c2 + 1) * a.cs + row] : mk<T>(T(0), T(0));
                if (kx == 0) {
                    zc[j * ln] = mk<T>(u1.x, u2.x);
                } else {
                    zc[j * ln + kx] = mk<T>(u1.x - u2.y, u1.y + u2.x);
                    zc[j * ln + n - kx] = mk<T>(u1.x + u2.y, u2.x - u1.y);
                }
            }
            __syncthreads();
            fft_into(c2, T(1));
        }
        T A0[9], D[9];
        for (int i = 0; i < d * d; ++i) {
            A0[i] = T(a.A0[i]);
            D[i] = T(a.D[i]);
        }
        double gs[9];
        for (int i = 0; i < 9; ++i) gs[i] = 0.0;
        for (int idx = threadIdx.x; idx < RP * n; idx += blockDim.x) {
            const int j = idx / n;
            const int x = idx - j * n;
            if (j >= nvr) continue;
            const long r = r0 + j;
            T am[9];
            if (a.nfield > 1) {
                sym_load<T>(g, a.gstride, r * n + x, d, am);
            } else {
                const T gg = g[r * n + x];
                for (int i = 0; i < d * d; ++i) am[i] = A0[i] + gg * D[i];
            }
            T f[3][3];
            for (int s2 = 0; s2 < d; ++s2)
                for (int b = 0; b < d; ++b) {
                    const int c = s2 * d + b;
                    const V zv = zbuf(c / 2)[j * ln + x];
                    f[s2][b] = ((c & 1) ? zv.y : zv.x) + (s2 == b ? T(1) : T(0));
                }
            for (int t = 0; t < d; ++t) {
                T af[3];
                for (int al = 0; al < d; ++al) {
                    T y = T(0);
                    for (int b = 0; b < d; ++b) y += am[al * d + b] * f[t][b];
                    af[al] = y;
                }
                for (int s2 = 0; s2 < d; ++s2) {
                    T dot = T(0);
                    for (int al = 0; al < d; ++al) dot += f[s2][al] * af[al];
                    gs[s2 * d + t] += dot;
                }
            }
        }
        for (int i = 0; i < d * d; ++i) {
            const double sum = block_sum(gs[i]);
            if (threadIdx.x == 0) a.partial[(long)blockIdx.x * d * d + i] = sum;
        }
        return;
    }

    // ---- spatial values ----
    if (zb && (a.mode == ROW_OPER || a.mode == ROW_GRAM || a.mode == ROW_C2R)) {
        const int nall = a.ncomp * RP;
        for (int idx = threadIdx.x; idx < nall * ln; idx += blockDim.x) Z[idx] = zero;
        __syncthreads();
        for (int idx = threadIdx.x; idx < nall * nh; idx += blockDim.x) {
            const int cj = idx / nh;  // c RP + j
            const int kx = idx - cj * nh;
            const int c = cj / RP;
            const int j = cj - c * RP;
            if (j >= nvp) continue;
            const int r1 = 2 * (pair0 + j);
            const int r2 = r1 + 1;
            const V u1 = data[(long)c * a.cs + (long)r1 * nh + kx];
            const V u2 = (r2 < a.nrows) ? data[(long)c * a.cs + (long)r2 * nh + kx] : mk<T>(T(0), T(0));
            V *zr = Z + (size_t)cj * ln;
            if (kx == 0) {
                zr[0] = mk<T>(u1.x, u2.x);
            } else {
                zr[kx] = mk<T>(u1.x - u2.y, u1.y + u2.x);
                zr[n - kx] = mk<T>(u1.x + u2.y, u2.x - u1.y);
            }
        }
        __syncthreads();
        const V *res = fft_lds<T, true, P13>(Z, S, a.f, nall, tw, T(1));
        if (res != Z) {
            for (int idx = threadIdx.x; idx < nall * ln; idx += blockDim.x) Z[idx] = res[idx];
            __syncthreads();
        }
    } else if (a.mode == ROW_OPER || a.mode == ROW_GRAM || a.mode == ROW_C2R) {
        for (int c = 0; c < a.ncomp; ++c) {
            V *zc = zbuf(c);
            for (int idx = threadIdx.x; idx < RP * ln; idx += blockDim.x) zc[idx] = zero;
            __syncthreads();
            for (int idx = threadIdx.x; idx < RP * nh; idx += blockDim.x) {
                const int j = idx / nh;
                const int kx = idx - j * nh;
                if (j >= nvp) continue;
                const int r1 = 2 * (pair0 + j);
                const int r2 = r1 + 1;
                const V u1 = data[(long)c * a.cs + (long)r1 * nh + kx];
                const V u2 = (r2 < a.nrows) ? data[(long)c * a.cs + (long)r2 * nh + kx] : mk<T>(T(0), T(0));
                if (kx == 0) {
                    zc[j * ln] = mk<T>(u1.x, u2.x);
                } else {
                    zc[j * ln + kx] = mk<T>(u1.x - u2.y, u1.y + u2.x);
                    zc[j * ln + n - kx] = mk<T>(u1.x + u2.y, u2.x - u1.y);
                }
            }
            __syncthreads();
            fft_into(c, T(1));
        }
    } else if (a.mode == ROW_R2C) {
        const T *rin = reinterpret_cast<const T *>(a.real_in);
        V *zc = zbuf(0);
        for (int idx = threadIdx.x; idx < RP * n; idx += blockDim.x) {
            const int j = idx / n;
            const int x = idx - j * n;
            V v = zero;
            if (j < nvp) {
                const int r1 = 2 * (pair0 + j);
                const int r2 = r1 + 1;
                v.x = map_voxel<T>(rin[(long)r1 * a.real_stride + x], a.imgmap, a.vmax);
                v.y = (r2 < a.nrows) ? map_voxel<T>(rin[(long)r2 * a.real_stride + x], a.imgmap, a.vmax) : T(0);
            }
            zc[j * ln + x] = v;
        }
        __syncthreads();
    }

    // ---- pointwise work ----
    if (a.mode == ROW_OPER || a.mode == ROW_RHS) {
        T A0[9], D[9], E[3];
        for (int i = 0; i < d * d; ++i) {
            A0[i] = T(a.A0[i]);
            D[i] = T(a.D[i]);
        }
        for (int i = 0; i < 3; ++i) E[i] = T(a.E[i]);
        double load = 0.0, work = 0.0;
        for (int idx = threadIdx.x; idx < RP * n; idx += blockDim.x) {
            const int j = idx / n;
            const int x = idx - j * n;
            if (j >= nvp) continue;
            const int r1 = 2 * (pair0 + j);
            const int r2 = r1 + 1;
            const bool v2 = r2 < a.nrows;
            T m1[9], m2[9];
            if (a.nfield > 1) {
                sym_load<T>(g, a.gstride, (long)r1 * n + x, d, m1);
                if (v2)
                    sym_load<T>(g, a.gstride, (long)r2 * n + x, d, m2);
                else
                    for (int i = 0; i < d * d; ++i) m2[i] = T(0);
            } else {
                const T g1 = g[(long)r1 * n + x];
                const T g2 = v2 ? g[(long)r2 * n + x] : T(0);
                for (int i = 0; i < d * d; ++i) {
                    m1[i] = A0[i] + g1 * D[i];
                    m2[i] = A0[i] + g2 * D[i];
                }
            }
            T e1[3], e2[3];
            for (int b = 0; b < d; ++b) {
                if (a.mode == ROW_OPER) {
                    const V zv = zbuf(b)[j * ln + x];
                    e1[b] = zv.x;
                    e2[b] = zv.y;
                } else {
                    e1[b] = E[b];
                    e2[b] = v2 ? E[b] : T(0);
                }
            }
            for (int al = 0; al < d; ++al) {
                T y1 = T(0), y2 = T(0);
                for (int b = 0; b < d; ++b) {
                    y1 += m1[al * d + b] * e1[b];
                    y2 += m2[al * d + b] * e2[b];
                }
                zbuf(al)[j * ln + x] = mk<T>(y1, y2);
                load += (double)y1 * y1 + (double)y2 * y2;
                if (a.mode == ROW_RHS) work += ((double)y1 + (double)y2) * a.E[al];
            }
        }
        __syncthreads();
        if (a.mode == ROW_RHS) {
            const double s = block_sum(load);
            const double s2 = block_sum(work);
            if (threadIdx.x == 0) {
                a.partial[blockIdx.x] = s;
                if (a.partial2 != nullptr) a.partial2[blockIdx.x] = s2;
            }
        }
    } else if (a.mode == ROW_GRAM) {
        // (A_M (E_s + e_s), E_t + e_t) summed over the rows' grid points
        T A0[9], D[9];
        for (int i = 0; i < d * d; ++i) {
            A0[i] = T(a.A0[i]);
            D[i] = T(a.D[i]);
        }
        double gs[9];
        for (int i = 0; i < 9; ++i) gs[i] = 0.0;
        for (int idx = threadIdx.x; idx < RP * n; idx += blockDim.x) {
            const int j = idx / n;
            const int x = idx - j * n;
            if (j >= nvp) continue;
            const int r1 = 2 * (pair0 + j);
            const int r2 = r1 + 1;
            for (int half = 0; half < 2; ++half) {
                const int r = half ? r2 : r1;
                if (r >= a.nrows) continue;
                T am[9];
                if (a.nfield > 1) {
                    sym_load<T>(g, a.gstride, (long)r * n + x, d, am);
                } else {
                    const T gg = g[(long)r * n + x];
                    for (int i = 0; i < d * d; ++i) am[i] = A0[i] + gg * D[i];
                }
                T f[3][3];
                for (int s = 0; s < d; ++s)
                    for (int b = 0; b < d; ++b) {
                        const V zv = zbuf(s * d + b)[j * ln + x];
                        f[s][b] = (half ? zv.y : zv.x) + (s == b ? T(1) : T(0));
                    }
                for (int t = 0; t < d; ++t) {
                    T af[3];
                    for (int al = 0; al < d; ++al) {
                        T y = T(0);
                        for (int b = 0; b < d; ++b) y += am[al * d + b] * f[t][b];
                        af[al] = y;
                    }
                    for (int s = 0; s < d; ++s) {
                        T dot = T(0);
                        for (int al = 0; al < d; ++al) dot += f[s][al] * af[al];
                        gs[s * d + t] += dot;
                    }
                }
            }
        }
        for (int i = 0; i < d * d; ++i) {
            const double s = block_sum(gs[i]);
            if (threadIdx.x == 0) a.partial[(long)blockIdx.x * d * d + i] = s;
        }
        return;
    } else if (a.mode == ROW_C2R) {
        T *rout = reinterpret_cast<T *>(a.real_out);
        const T scale = T(a.scale);
        for (int idx = threadIdx.x; idx < RP * n; idx += blockDim.x) {
            const int j = idx / n;
            const int x = idx - j * n;
            if (j >= nvp) continue;
            const int r1 = 2 * (pair0 + j);
            const int r2 = r1 + 1;
            const V zv = zbuf(0)[j * ln + x];
            rout[(long)r1 * a.real_stride + x] = zv.x * scale;
            if (r2 < a.nrows) rout[(long)r2 * a.real_stride + x] = zv.y * scale;
        }
        return;
    }

    // ---- forward transforms and Hermitian split ----
    const T half = T(a.scale) * T(0.5);
    if (zb) {
        const V *res = fft_lds<T, true, P13>(Z, S, a.f, nzc * RP, tw, T(-1));
        for (int idx = threadIdx.x; idx < nzc * RP * nh; idx += blockDim.x) {
            const int cj = idx / nh;
            const int kx = idx - cj * nh;
            const int c = cj / RP;
            const int j = cj - c * RP;
            if (j >= nvp) continue;
            const int r1 = 2 * (pair0 + j);
            const int r2 = r1 + 1;
            const V *zr = res + (size_t)cj * ln;
            const V w = zr[posmod(kx, n)];
            const V wm = zr[posmod(-kx, n)];
            data[(long)c * a.cs + (long)r1 * nh + kx] = mk<T>((w.x + wm.x) * half, (w.y - wm.y) * half);
            if (r2 < a.nrows)
                data[(long)c * a.cs + (long)r2 * nh + kx] = mk<T>((w.y + wm.y) * half, (wm.x - w.x) * half);
        }
        return;
    }
    for (int c = 0; c < nzc; ++c) {
        fft_into(c, T(-1));
        const V *zc = zbuf(c);
        for (int idx = threadIdx.x; idx < RP * nh; idx += blockDim.x) {
            const int j = idx / nh;
            const int kx = idx - j * nh;
            if (j >= nvp) continue;
            const int r1 = 2 * (pair0 + j);
            const int r2 = r1 + 1;
            const V w = zc[j * ln + posmod(kx, n)];
            const V wm = zc[j * ln + posmod(-kx, n)];
            data[(long)c * a.cs + (long)r1 * nh + kx] = mk<T>((w.x + wm.x) * half, (w.y - wm.y) * half);
            if (r2 < a.nrows)
                data[(long)c * a.cs + (long)r2 * nh + kx] = mk<T>((w.y + wm.y) * half, (wm.x - w.x) * half);
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// CG scalar and vector kernels (Remark CG; Saad Alg. 6.18).
// ---------------------------------------------------------------------------
// Sum of n partials in a fixed order: thread t adds entries t, t + blockDim,
// t + 2 blockDim, ... in turn, then block_sum; the loads of eight such steps
// are issued together (an entry past n adds an exact zero).
__device__ double sum_fixed(const double *part, int n) {
    constexpr int G = 8;
    double v = 0.0;
    for (int i0 = threadIdx.x; i0 < n; i0 += G * blockDim.x) {
        double t[G];
#pragma unroll
        for (int j = 0; j < G; ++j) {
            const int i = i0 + j * (int)blockDim.x;
            t[j] = i < n ? part[i] : 0.0;
        }
#pragma unroll
        for (int j = 0; j < G; ++j) v += t[j];
    }
    return block_sum(v);
}

// hist[0] = (r_0, r_0); hist[1] = the energy (A_M E, E) of the initial iterate
// e_0 = 0 (the Voigt entry), from the right-hand side pass's sums of (A_M E).E.
__device__ void cg_init(const InitArgs &a) {
    CgStatus *st = a.st;
    double *hist = a.hist;
    const double inv_mtot = a.inv_mtot, tol = a.tol, floor_rel = a.floor_rel, btol = a.btol;
    const int maxit = a.maxit;
    const double rr = sum_fixed(a.rr_part, a.n_rr);
    const double load = sum_fixed(a.load_part, a.n_load);
    const double work = a.work_part != nullptr ? sum_fixed(a.work_part, a.n_load) : 0.0;
    if (threadIdx.x == 0) {
        st->rr = rr;
        st->rr0 = rr;
        st->pq = 0.0;
        st->alpha = 0.0;
        st->beta = 0.0;
        st->tol2 = tol * tol;
        st->load2 = load;
        st->floor2 = floor_rel * floor_rel * load;
        st->iter = 0;
        st->maxit = maxit;
        st->energy = work * inv_mtot;
        st->dprev = 0.0;
        st->btol = btol;
        st->eAE = st->energy;
        st->ebest = st->energy;  // e_0 = 0: the kept copy starts as zero
        st->rrmin = rr;
        st->rrmin_it = 0;
        st->best_it = 0;
        st->stagnated = 0;
        st->ck_copy = 0;
        st->ck_restore = 0;
        st->breakdown = !isfinite(rr) || !isfinite(load);
        st->converged = (rr == 0.0 || rr <= st->floor2) && !st->breakdown;
        st->done = st->converged || st->breakdown || maxit <= 0;
        if (hist != nullptr) {
            hist[0] = rr;
            hist[1] = st->energy;
        }
    }
}

__global__ __launch_bounds__(kThreads) void cg_init_kernel(InitArgs a) { cg_init(a); }
__global__ __launch_bounds__(kThreads) void cg_init_multi_kernel(const InitArgs *a) { cg_init(a[blockIdx.x]); }

// Warm start from an admissible initial iterate x0 (Remark CG: CG from an
// initial approximation in the minimisation space): r_0 = b - K x0 with r
// holding b and q = K x0 on entry; partial sums of (r_0, r_0), (b, x0) and
// (r_0, x0) in the weights of the half-spectrum storage.
template <typename T>
__global__ __launch_bounds__(kThreads) void warm_residual_kernel(UpdArgs a, double *part_rr, double *part_bx,
                                                                 double *part_rx) {
    Vt<T> *r = reinterpret_cast<Vt<T> *>(a.r);
    const Vt<T> *x = reinterpret_cast<const Vt<T> *>(a.x);
    const Vt<T> *q = reinterpret_cast<const Vt<T> *>(a.q);
    double prr = 0.0, pbx = 0.0, prx = 0.0;
    const long total = a.n_per_comp * a.nc;
    for (long idx = blockIdx.x * (long)kThreads + threadIdx.x; idx < total; idx += (long)a.nblocks * kThreads) {
        const long c = idx / a.n_per_comp;
        const long i = idx - c * a.n_per_comp;
        const long off = c * a.cs + i;
        const Vt<T> bv = r[off], qv = q[off], xv = x[off];
        Vt<T> rv = bv;
        rv.x -= qv.x;
        rv.y -= qv.y;
        r[off] = rv;
        const double w = (i % a.Nh) == 0 ? 1.0 : 2.0;
        prr += w * ((double)rv.x * rv.x + (double)rv.y * rv.y);
        pbx += w * ((double)bv.x * xv.x + (double)bv.y * xv.y);
        prx += w * ((double)rv.x * xv.x + (double)rv.y * xv.y);
    }
    const double s1 = block_sum(prr);
    const double s2 = block_sum(pbx);
    const double s3 = block_sum(prx);
    if (threadIdx.x == 0) {
        part_rr[blockIdx.x] = s1;
        part_bx[blockIdx.x] = s2;
        part_rx[blockIdx.x] = s3;
    }
}

// Energy at x0: (A(E + x0), E + x0) = (A E, E) + 2 phi(x0), phi(x) =
// (K x, x) / 2 - (b, x), and (K x0, x0) = (b - r_0, x0).
__global__ __launch_bounds__(kThreads) void cg_init_warm_kernel(CgStatus *st, const double *part_rr,
                                                                const double *part_bx, const double *part_rx,
                                                                int nparts, const double *scal, double mtot,
                                                                double tol, double floor_rel, int maxit, double btol,
                                                                double *hist) {
    const double rr = sum_fixed(part_rr, nparts);
    const double bx = sum_fixed(part_bx, nparts);
    const double rx = sum_fixed(part_rx, nparts);
    if (threadIdx.x == 0) {
        const double bb = scal[0];
        const double load = scal[1];
        st->rr = rr;
        st->rr0 = bb;
        st->pq = 0.0;
        st->alpha = 0.0;
        st->beta = 0.0;
        st->tol2 = tol * tol;
        st->load2 = load;
        st->floor2 = floor_rel * floor_rel * load;
        st->iter = 0;
        st->maxit = maxit;
        st->energy = scal[2] / mtot - bx - rx;
        st->dprev = 0.0;
        st->btol = btol;
        st->eAE = scal[2] / mtot;
        st->ebest = st->energy;  // the kept copy starts as the initial iterate
        st->rrmin = rr;
        st->rrmin_it = 0;
        st->best_it = 0;
        st->stagnated = 0;
        st->ck_copy = 0;
        st->ck_restore = 0;
        st->breakdown = !isfinite(rr) || !isfinite(load) || !isfinite(bb);
        st->converged = (rr == 0.0 || rr <= st->tol2 * bb || rr <= st->floor2) && !st->breakdown;
        st->done = st->converged || st->breakdown || maxit <= 0;
        if (hist != nullptr) {
            hist[0] = rr;
            hist[1] = st->energy;
        }
    }
}

// Prolongation of the coefficients of a coarse solve (grid Nc) to a fine one
// (grid Nf): the trigonometric polynomial is kept (Fourier zero padding), so
// the entries of frequencies k in Z_Nc move and all others are zero.  Storage
// [c][k1][k2][k3 >= 0] (2D: [c][k1][k2 >= 0]) with wrapped indices.
template <typename TS, typename TD>
__global__ __launch_bounds__(kThreads) void prolong_kernel(const Vt<TS> *src, Vt<TD> *dst, int d, int nc, int f1,
                                                           int f2, int f3h, int c1, int c2, int c3h) {
    const long nsf = (long)f1 * f2 * f3h;  // 2D: f2 = 1
    const long nsc = (long)c1 * c2 * c3h;
    const long total = nsf * nc;
    for (long idx = blockIdx.x * (long)kThreads + threadIdx.x; idx < total; idx += (long)gridDim.x * kThreads) {
        const long c = idx / nsf;
        long rem = idx - c * nsf;
        const int i3 = (int)(rem % f3h);
        rem /= f3h;
        const int i2 = (int)(rem % f2);
        const int i1 = (int)(rem / f2);
        const int k1 = wrapi(i1, f1);
        const int k2 = d == 3 ? wrapi(i2, f2) : 0;
        const bool in = (k1 >= -(c1 / 2) && k1 < (c1 + 1) / 2) && (d == 2 || (k2 >= -(c2 / 2) && k2 < (c2 + 1) / 2)) &&
                        i3 < c3h;
        Vt<TD> v;
        v.x = TD(0);
        v.y = TD(0);
        if (in) {
            const long j = ((long)posmod(k1, c1) * c2 + (d == 3 ? posmod(k2, c2) : 0)) * c3h + i3;
            const Vt<TS> u = src[c * nsc + j];
            v.x = TD(u.x);
            v.y = TD(u.y);
        }
        dst[idx] = v;
    }
}




__global__ void fill_zero_kernel(unsigned int *p, size_t nwords) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < nwords; i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

__global__ __launch_bounds__(kThreads) void vec_ops_kernel(VecOps v) {
    const VecOps::Op &o = v.op[blockIdx.y];
    unsigned int *d = static_cast<unsigned int *>(o.dst);
    const unsigned int *s = static_cast<const unsigned int *>(o.src);
    for (size_t i = blockIdx.x * (size_t)kThreads + threadIdx.x; i < o.words; i += (size_t)gridDim.x * kThreads)
        d[i] = s != nullptr ? s[i] : 0u;
}

__global__ void f2d_kernel(double *dst, const float *src, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        dst[i] = (double)src[i];
}

__global__ void d2f_kernel(float *dst, const double *src, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        dst[i] = (float)src[i];
}

// out[v] = sum_i part[i * nvals + v] in a fixed order (work-group v).
__global__ __launch_bounds__(kThreads) void sum_partials_kernel(double *out, const double *part, int nparts,
                                                                int nvals) {
    const int v = blockIdx.x;
    double s = 0.0;
    for (int i = threadIdx.x; i < nparts; i += blockDim.x) s += part[(long)i * nvals + v];
    s = block_sum(s);
    if (threadIdx.x == 0) out[v] = s;
}

// Fourier coefficients on the half grid of Z_{L} (L = 2N-1): entry
// (n_1, [n_2,] n_3 >= 0) = w0 [n = 0] + sum_i w_i exp(-2 pi i n.c_i) fhat_i(n),
// with fhat of the box prod_a h_a sinc(h_a n_a) or of the disc
// r J_1(2 pi r |n|)/|n| (pi r^2 at n = 0)  (eq. char_func_Four, eq. inclcomp_formula).
__global__ __launch_bounds__(kThreads) void incl_coeff_kernel(double2 *out, int d, int L1, int L2, int Lh,
                                                              const InclDev *incl, int n_incl, double w0) {
    const long total = (d == 3 ? (long)L1 * L2 * Lh : (long)L1 * Lh);
    for (long idx = blockIdx.x * (long)blockDim.x + threadIdx.x; idx < total; idx += (long)gridDim.x * blockDim.x) {
        int n1, n2, n3;
        if (d == 3) {
            n3 = (int)(idx % Lh);
            n2 = wrapi((int)((idx / Lh) % L2), L2);
            n1 = wrapi((int)(idx / ((long)Lh * L2)), L1);
        } else {
            n3 = 0;
            n2 = (int)(idx % Lh);
            n1 = wrapi((int)(idx / Lh), L1);
        }
        double re = (n1 == 0 && n2 == 0 && n3 == 0) ? w0 : 0.0, im = 0.0;
        for (int i = 0; i < n_incl; ++i) {
            const InclDev &q = incl[i];
            double f;
            if (q.shape == 0) {
                f = q.h[0] * sinc_pi(q.h[0] * n1) * q.h[1] * sinc_pi(q.h[1] * n2);
                if (d == 3) f *= q.h[2] * sinc_pi(q.h[2] * n3);
            } else {
                const double kn = sqrt((double)n1 * n1 + (double)n2 * n2);
                const double r = q.h[0];
                f = kn == 0.0 ? M_PI * r * r : r * j1(2.0 * M_PI * r * kn) / kn;
            }
            const double arg = -2.0 * ((double)n1 * q.c[0] + (double)n2 * q.c[1] + (d == 3 ? (double)n3 * q.c[2] : 0.0));
            double sv, cv;
            sincospi(arg, &sv, &cv);
            re += q.w * f * cv;
            im += q.w * f * sv;
        }
        out[idx] = make_double2(re, im);
    }
}


// ---- multi-problem CG kernels (one problem per work-group for the scalar one) ----
__global__ __launch_bounds__(kThreads) void cg_check_multi_kernel(const CgItem *__restrict__ items) {
    const CgItem &it = items[blockIdx.x];
    CgStatus *st = it.st;
    if (!st->done) {
        const double rr = sum_fixed(it.rr_part, it.nrr);
        if (threadIdx.x == 0) {
            const int iter = st->iter + 1;
            st->iter = iter;
            if (it.hist != nullptr && iter < it.hist_cap) {
                it.hist[2 * iter] = rr;
                it.hist[2 * iter + 1] = st->alpha;
            }
            if (!isfinite(rr)) {
                st->breakdown = 1;
                st->done = 1;
            } else {
                // energy of the new iterate: one CG step lowers it by
                // alpha_k (r_{k-1}, r_{k-1})
                const double dstep = st->alpha * st->rr;
                st->energy -= dstep;
                st->beta = rr / st->rr;
                st->rr = rr;
                if (rr < st->rrmin) {
                    st->rrmin = rr;
                    st->rrmin_it = iter;
                }
                if (rr <= st->tol2 * st->rr0 || rr <= st->floor2) {
                    st->converged = 1;
                    st->done = 1;
                } else if (st->btol > 0.0 && iter >= 2 && st->dprev > 0.0 &&
                           dstep <= st->btol * fabs(st->energy) *
                                        (1.0 - fmin(fmax(dstep / st->dprev, 0.0), 0.99))) {
                    // bound test: the remaining decrease, estimated from the
                    // ratio q of the last two steps as dstep q / (1 - q), is
                    // below btol times the bound entry
                    st->converged = 1;
                    st->done = 1;
                } else if (iter >= st->maxit) {
                    st->done = 1;
                }
                st->dprev = dstep;
            }
        }
    }
    if (it.mirror != nullptr && threadIdx.x == 0) *it.mirror = *st;
}

// CG update: kUpdPer elements per thread in one pass (the grid, and with it
// the reduction order, depends only on the problem size).  Every work-group
// sums the (p, K p) partials of the projection pass itself, in one fixed
// order, while its vector loads are in flight, and forms alpha = (r, r) /
// (p, K p); work-group 0 records pq and alpha (or a breakdown) in the status.
constexpr int kUpdPer = 2;
template <typename T>
__global__ __launch_bounds__(kThreads) void cg_update_multi_kernel(const UpdArgs *__restrict__ ua,
                                                                   const int *__restrict__ woff, int np) {
    constexpr int U = kUpdPer;
    __shared__ double bcast;
    int lb;
    const UpdArgs &a = ua[find_problem(woff, np, &lb)];
    CgStatus *st = a.st;
    if (st->done) return;
    const double rr = st->rr;
    auto *x = gbl(reinterpret_cast<Vt<T> *>(a.x));
    auto *r = gbl(reinterpret_cast<Vt<T> *>(a.r));
    const auto *p = gbl(reinterpret_cast<const Vt<T> *>(a.p));
    const auto *q = gbl(reinterpret_cast<const Vt<T> *>(a.q));
    const int npc = (int)a.n_per_comp;
    const int total = npc * a.nc;
    // all loads of the thread's U elements in flight together
    T xx[U], xy[U], rx[U], ry[U], px[U], py[U], qx[U], qy[U];
    long off[U];
    int ii[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
        const int idx = lb * (kThreads * U) + j * kThreads + threadIdx.x;
        const int c = idx / npc;
        ii[j] = idx - c * npc;
        off[j] = idx < total ? (long)c * a.cs + ii[j] : -1L;
        const long o = off[j] < 0 ? 0L : off[j];
        const Vt<T> xv = gld(x + o), rv = gld(r + o), pv = gld(p + o), qv = gld(q + o);
        xx[j] = xv.x;
        xy[j] = xv.y;
        rx[j] = rv.x;
        ry[j] = rv.y;
        px[j] = pv.x;
        py[j] = pv.y;
        qx[j] = qv.x;
        qy[j] = qv.y;
    }
    // the other shifts' contributions to K p, added in shift order
    for (int sh = 1; sh < a.nq; ++sh) {
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const long o = off[j] < 0 ? 0L : off[j];
            const Vt<T> qv = gld(q + sh * a.q_ss + o);
            qx[j] += qv.x;
            qy[j] += qv.y;
        }
    }
    const double pq = sum_fixed(a.pq_part, a.npq);
    if (threadIdx.x == 0) bcast = pq;
    __syncthreads();
    const double pqa = bcast;
    const bool bad = !(pqa > 0.0) || !isfinite(pqa);
    const double alpha_d = bad ? 0.0 : rr / pqa;
    if (lb == 0 && threadIdx.x == 0) {
        st->pq = pqa;
        if (bad) {
            // the material is SPD (validated when it is set), so with FP32
            // iterates a finite (p, K p) <= 0 after the first step is rounding
            // that has overtaken the iteration: a stall, and the best iterate
            // is kept; in FP64, or at the first step, the operator is at fault
            if (sizeof(T) == 4 && isfinite(pqa) && st->iter > 0)
                st->stagnated = 1;
            else
                st->breakdown = 1;
            st->done = 1;
        } else {
            st->alpha = alpha_d;
        }
    }
    if (bad) return;
    const T alpha = T(alpha_d);
    double part = 0.0;
#pragma unroll
    for (int j = 0; j < U; ++j) {
        if (off[j] < 0) continue;
        const T nxx = xx[j] + alpha * px[j], nxy = xy[j] + alpha * py[j];
        const T nrx = rx[j] - alpha * qx[j], nry = ry[j] - alpha * qy[j];
        gst(x + off[j], mk<T>(nxx, nxy));
        gst(r + off[j], mk<T>(nrx, nry));
        const double w = (ii[j] % a.Nh) == 0 ? 1.0 : 2.0;
        part += w * ((double)nrx * nrx + (double)nry * nry);
    }
    const double s = block_sum(part);
    if (threadIdx.x == 0) a.partial[lb] = s;
}

// ---------------------------------------------------------------------------
// Whole 2D CG solves, one work-group each (small double grids).  The CG
// vectors stay in registers (each thread owns coefficients idx = tid + 1024 j
// of the N0 x Nh half spectrum); the operator of Algorithm 2 runs on one
// complex M0 x M1 grid in LDS: the two components y_0, y_1 of the gradient
// field (real on the grid) are packed as z = y_0 + i y_1, so that
//   Z(k) = Y_0(k) + i Y_1(k),  Y_c(k) = i t_c(k) p(k)  (k_1 >= 0 stored;
//   Z(-k) = conj(Y_0(k)) + i conj(Y_1(k)) from the Hermitian symmetry),
// an inverse 2D DFT gives z on the grid, the material acts on (Re z, Im z) at
// every point, a forward 2D DFT gives Z', and
//   Y'_0(k) = (Z'(k) + conj(Z'(-k))) / 2,  Y'_1(k) = (Z'(k) - conj(Z'(-k))) / 2i
// feed the projection q(k) = -i scale sum_c t_c(k) Y'_c(k).  The CG update and
// the stopping test (as cg_update_multi_kernel and cg_check_multi_kernel,
// with work-group sums in a fixed order) follow in the same work-group, so a
// launch runs many iterations with no kernel boundary between them.
// ---------------------------------------------------------------------------
//
// Two forms share the kernel: lengths of 81 or 125 points known at compile
// time (FI0, FI1 their indices), and any 3,5,7-smooth lengths taken from the
// arguments (FI0 = -1) for the other grids that fit; the latter use 256 or 512
// threads on small grids, where a barrier of fewer waves costs less than the
// idle lanes save.
constexpr int kSoloNT = 1024;
template <typename T>
constexpr size_t solo_lds_bytes_t(int m0, int m1) {
    return sizeof(Vt<T>) * ((size_t)m0 * m1 + m0 + m1 + (m0 + 1) / 2);
}

// fixed-order sum over the NT threads (shuffle tree per wave, then the
// waves in turn by thread 0), broadcast to every thread
template <int NT>
__device__ __forceinline__ double solo_sum(double v, double *red) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) red[wave] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < NT / 64; ++w) s += red[w];
        red[NT / 64] = s;
    }
    __syncthreads();
    return red[NT / 64];
}

// x / d for x < 2^32 / d, with m = floor(2^32 / d) + 1 (0 stands for d = 1)
__device__ __forceinline__ int solo_div(int x, unsigned m) { return m == 0 ? x : (int)__umulhi((unsigned)x, m); }

// Most butterflies of radix R per thread of an in-place stage: their values
// wait in registers for the barrier.
constexpr int solo_per(int R, bool fp64) {
    return R == 3 ? (fp64 ? 3 : 6) : R == 5 ? (fp64 ? 2 : 4) : R == 7 ? (fp64 ? 2 : 3) : R <= 15 ? (fp64 ? 1 : 2) : 1;
}

// One in-place stage of radix R along axis 0 (COL: the NA non-zero columns of
// the [.][M1] grid) or axis 1 (rows), over nb transforms.
template <typename T, int R, bool COL, int NT>
__device__ __forceinline__ void solo_stage(Vt<T> *X, const Vt<T> *tw, const SoloStage &g, int M1, int nb, int Nh,
                                           unsigned mNA, T sg) {
    constexpr int PER = solo_per(R, sizeof(T) == 8);
    const int TQ = g.TQ, P = g.P;
    const int tot = TQ * nb;
    Vt<T> u[PER][R];
    int base[PER], k[PER], i[PER];
#pragma unroll
    for (int t = 0; t < PER; ++t) {
        const int idx = threadIdx.x + t * NT;
        if (idx >= tot) break;
        if (COL) {
            i[t] = solo_div(idx, mNA);
            const int c = idx - i[t] * nb;
            base[t] = c < Nh ? c : c + (M1 - nb);
        } else {
            const int b = solo_div(idx, g.mTQ);
            i[t] = idx - b * TQ;
            base[t] = b * M1;
        }
        k[t] = i[t] - solo_div(i[t], g.mP) * P;
#pragma unroll
        for (int q = 0; q < R; ++q) u[t][q] = X[base[t] + (i[t] + q * TQ) * (COL ? M1 : 1)];
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < PER; ++t) {
        const int idx = threadIdx.x + t * NT;
        if (idx >= tot) break;
        if (P > 1) {
#pragma unroll
            for (int q = 1; q < R; ++q) {
                Vt<T> w = tw[(q - 1) * P + k[t]];
                w.y *= -sg;
                u[t][q] = cmul(u[t][q], w);
            }
        }
        dftn<T, R>(u[t], sg);
        const int j = (i[t] - k[t]) * R + k[t];
#pragma unroll
        for (int q = 0; q < R; ++q) X[base[t] + (j + q * P) * (COL ? M1 : 1)] = u[t][q];
    }
    __syncthreads();
}

template <typename T, bool COL, int NT>
__device__ __forceinline__ void solo_fft(Vt<T> *X, const Vt<T> *tw, const SoloArgs &a, int nb, T sg) {
    for (int s = 0; s < a.nst[COL ? 0 : 1]; ++s) {
        const SoloStage &g = a.stg[COL ? 0 : 1][s];
        const Vt<T> *t = tw + g.tw;
        switch (g.R) {
            case 3: solo_stage<T, 3, COL, NT>(X, t, g, a.M1, nb, a.Nh, a.mNA, sg); break;
            case 5: solo_stage<T, 5, COL, NT>(X, t, g, a.M1, nb, a.Nh, a.mNA, sg); break;
            case 7: solo_stage<T, 7, COL, NT>(X, t, g, a.M1, nb, a.Nh, a.mNA, sg); break;
            case 9: solo_stage<T, 9, COL, NT>(X, t, g, a.M1, nb, a.Nh, a.mNA, sg); break;
            case 15: solo_stage<T, 15, COL, NT>(X, t, g, a.M1, nb, a.Nh, a.mNA, sg); break;
            default: solo_stage<T, 25, COL, NT>(X, t, g, a.M1, nb, a.Nh, a.mNA, sg); break;
        }
    }
}

// coefficients per thread: the half spectrum of the compile-time grid, or two
// (1024 threads) and one otherwise
constexpr int solo_cpt(int fi0, int fi1, int nt) {
    if (fi0 < 0) return nt == 1024 ? 2 : 1;
    return ((kFastSched[fi0].n + 1) / 2 * ((kFastSched[fi1].n + 3) / 4) + nt - 1) / nt;
}
template <typename T, int FI0, int FI1, int NT>
__global__ __launch_bounds__(NT) void solo2d_kernel(const SoloArgs *__restrict__ sa, int niter) {
    using V = Vt<T>;
    constexpr bool ANY = FI0 < 0;  // lengths from the arguments
    constexpr int CPT = solo_cpt(FI0, FI1, NT);
    const SoloArgs &a = sa[blockIdx.x];
    const int M0 = ANY ? a.M0 : kFastSched[ANY ? 0 : FI0].n, M1 = ANY ? a.M1 : kFastSched[ANY ? 0 : FI1].n;
    __shared__ CgStatus S;
    __shared__ double red[NT / 64 + 1];
    extern __shared__ __align__(16) unsigned char smem_raw[];
    V *Z = reinterpret_cast<V *>(smem_raw);  // [M0][M1]
    V *tw0 = Z + M0 * M1;                    // stage twiddles of axis 0
    V *tw1 = tw0 + M0;                       // and of axis 1
    V *P0 = tw1 + M1;                        // p at k_2 = 0, by stored index of k_1
    if (threadIdx.x == 0) S = *a.st;
    {
        const auto *t0 = gbl(reinterpret_cast<const V *>(a.tw) + a.tw0);
        const auto *t1 = gbl(reinterpret_cast<const V *>(a.tw) + a.tw1);
        for (int i = threadIdx.x; i < M0 - 1; i += NT) tw0[i] = gld(t0 + i);
        for (int i = threadIdx.x; i < M1 - 1; i += NT) tw1[i] = gld(t1 + i);
    }
    const int N0 = a.N0, Nh = a.Nh;
    const int ns = N0 * Nh;
    auto *gx = gbl(reinterpret_cast<V *>(a.x));
    auto *gr = gbl(reinterpret_cast<V *>(a.r));
    auto *gp = gbl(reinterpret_cast<V *>(a.p));
    T xr[CPT], xi[CPT], rr_[CPT], ri[CPT], pr[CPT], pi_[CPT], t0[CPT], t1[CPT], wgt[CPT];
    int zp[CPT], zm[CPT], lz[CPT];
    bool own[CPT], pos1[CPT];
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
        const int idx = threadIdx.x + j * NT;
        own[j] = idx < ns;
        const int id = own[j] ? idx : 0;
        const int l = ANY ? solo_div(id, a.mNh) : id / Nh;
        const int k1 = id - l * Nh;
        const int k0 = wrapi(l, N0);
        T tb[2][3];
        const int nt = basis<T>(2, a.kind, k0, k1, 0, tb);
        t0[j] = nt ? tb[0][0] : T(0);
        t1[j] = nt ? tb[0][1] : T(0);
        pos1[j] = k1 > 0;
        lz[j] = k1 == 0 ? l : -1;
        wgt[j] = k1 == 0 ? T(1) : T(2);
        zp[j] = posmod(k0, M0) * M1 + k1;
        zm[j] = posmod(-k0, M0) * M1 + (k1 == 0 ? 0 : M1 - k1);
        const V vx = gld(gx + id), vr = gld(gr + id), vp = gld(gp + id);
        xr[j] = vx.x;
        xi[j] = vx.y;
        rr_[j] = vr.x;
        ri[j] = vr.y;
        pr[j] = vp.x;
        pi_[j] = vp.y;
    }
    const auto *g = gbl(reinterpret_cast<const T *>(a.g));
    const T A00 = T(a.A0[0]), A01 = T(a.A0[1]), A11 = T(a.A0[3]);
    const T D00 = T(a.D[0]), D01 = T(a.D[1]), D11 = T(a.D[3]);
    const T scale = T(a.scale);
    __syncthreads();
    for (int it = 0; it < niter && !S.done; ++it) {
        // p = r + beta p (beta = 0 at the first step of a solve)
        const T beta = T(S.beta);
#pragma unroll
        for (int j = 0; j < CPT; ++j) {
            pr[j] = rr_[j] + beta * pr[j];
            pi_[j] = ri[j] + beta * pi_[j];
            if (own[j] && lz[j] >= 0) P0[lz[j]] = mk<T>(pr[j], pi_[j]);
        }
        for (int i = threadIdx.x; i < M0 * M1; i += NT) Z[i] = mk<T>(T(0), T(0));
        __syncthreads();
#pragma unroll
        for (int j = 0; j < CPT; ++j) {
            if (!own[j]) continue;
            // at k_2 = 0 the stored pair p(k_1, 0), p(-k_1, 0) enters through its
            // Hermitian part (p(k) + conj(p(-k))) / 2, the part a real field has
            // (as the per-pass kernels, whose real transform along the last
            // axis keeps the real part there); the rest, rounding of the
            // right-hand side, must not reach the field
            T px = pr[j], py = pi_[j];
            if (lz[j] >= 0) {
                const V pm = P0[lz[j] == 0 ? 0 : N0 - lz[j]];
                px = (px + pm.x) * T(0.5);
                py = (py - pm.y) * T(0.5);
            }
            // Y_c = i t_c p
            const T y0x = -t0[j] * py, y0y = t0[j] * px;
            const T y1x = -t1[j] * py, y1y = t1[j] * px;
            Z[zp[j]] = mk<T>(y0x - y1y, y0y + y1x);
            if (pos1[j]) Z[zm[j]] = mk<T>(y0x + y1y, y1x - y0y);
        }
        __syncthreads();
        // columns: only the N_2 = (M_2 + 1) / 2 non-zero ones (zero-padded
        // frequencies stay zero, and only they are read back after the
        // forward transform)
        if constexpr (ANY) {
            solo_fft<T, true, NT>(Z, tw0, a, 2 * Nh - 1, T(1));
            solo_fft<T, false, NT>(Z, tw1, a, M0, T(1));
        } else {
            constexpr int C0 = kFastSched[FI0].n, C1 = kFastSched[FI1].n;
            fft_ip<T, FI0, 0, 1, 0, C1, false, NT, (C1 + 1) / 2>(Z, tw0, T(1));
            fft_ip<T, FI1, 0, 1, 0, C0, true, NT>(Z, tw1, T(1));
        }
        if (a.nfield == 1) {
            for (int i = threadIdx.x; i < M0 * M1; i += NT) {
                const V z = Z[i];
                const T gv = g[i];
                const T a00 = A00 + gv * D00, a01 = A01 + gv * D01, a11 = A11 + gv * D11;
                Z[i] = mk<T>(a00 * z.x + a01 * z.y, a01 * z.x + a11 * z.y);
            }
        } else {
            for (int i = threadIdx.x; i < M0 * M1; i += NT) {
                const V z = Z[i];
                const T a00 = g[i], a01 = g[a.gstride + i], a11 = g[2 * a.gstride + i];
                Z[i] = mk<T>(a00 * z.x + a01 * z.y, a01 * z.x + a11 * z.y);
            }
        }
        __syncthreads();
        if constexpr (ANY) {
            solo_fft<T, false, NT>(Z, tw1, a, M0, T(-1));
            solo_fft<T, true, NT>(Z, tw0, a, 2 * Nh - 1, T(-1));
        } else {
            constexpr int C0 = kFastSched[FI0].n, C1 = kFastSched[FI1].n;
            fft_ip<T, FI1, 0, 1, 0, C0, true, NT>(Z, tw1, T(-1));
            fft_ip<T, FI0, 0, 1, 0, C1, false, NT, (C1 + 1) / 2>(Z, tw0, T(-1));
        }
        // projection q = -i scale sum_c t_c Y'_c and the partial of (p, q)
        T qr[CPT], qi[CPT];
        double part = 0.0;
#pragma unroll
        for (int j = 0; j < CPT; ++j) {
            qr[j] = qi[j] = T(0);
            if (!own[j]) continue;
            const V zk = Z[zp[j]], zn = Z[zm[j]];
            const T h = T(0.5);
            const T y0x = (zk.x + zn.x) * h, y0y = (zk.y - zn.y) * h;
            const T y1x = (zk.y + zn.y) * h, y1y = (zn.x - zk.x) * h;
            const T s0 = t0[j] * scale, s1 = t1[j] * scale;
            qr[j] = s0 * y0y + s1 * y1y;
            qi[j] = -(s0 * y0x + s1 * y1x);
            part += (double)wgt[j] * ((double)pr[j] * (double)qr[j] + (double)pi_[j] * (double)qi[j]);
        }
        const double pq = solo_sum<NT>(part, red);
        const bool bad = !(pq > 0.0) || !isfinite(pq);
        if (threadIdx.x == 0) {
            S.pq = pq;
            if (bad) {
                // as the update pass: with FP32 iterates a finite (p, K p) <= 0
                // after the first step is a stall, otherwise a breakdown
                if (sizeof(T) == 4 && isfinite(pq) && S.iter > 0)
                    S.stagnated = 1;
                else
                    S.breakdown = 1;
                S.done = 1;
            } else {
                S.alpha = S.rr / pq;
            }
        }
        if (bad) break;  // uniform: pq is the same in every thread
        const double alpha_d = S.rr / pq;
        const T alpha = T(alpha_d);
        double part2 = 0.0;
#pragma unroll
        for (int j = 0; j < CPT; ++j) {
            if (!own[j]) continue;
            xr[j] = xr[j] + alpha * pr[j];
            xi[j] = xi[j] + alpha * pi_[j];
            rr_[j] = rr_[j] - alpha * qr[j];
            ri[j] = ri[j] - alpha * qi[j];
            part2 += (double)wgt[j] * ((double)rr_[j] * rr_[j] + (double)ri[j] * ri[j]);
        }
        const double rr = solo_sum<NT>(part2, red);
        if (threadIdx.x == 0) {
            // the stopping test of cg_check_multi_kernel
            const int iter = S.iter + 1;
            S.iter = iter;
            if (a.hist != nullptr && iter < a.hist_cap) {
                a.hist[2 * iter] = rr;
                a.hist[2 * iter + 1] = S.alpha;
            }
            if (!isfinite(rr)) {
                S.breakdown = 1;
                S.done = 1;
            } else {
                const double dstep = S.alpha * S.rr;
                S.energy -= dstep;
                S.beta = rr / S.rr;
                S.rr = rr;
                if (rr < S.rrmin) {
                    S.rrmin = rr;
                    S.rrmin_it = iter;
                }
                if (rr <= S.tol2 * S.rr0 || rr <= S.floor2) {
                    S.converged = 1;
                    S.done = 1;
                } else if (S.btol > 0.0 && iter >= 2 && S.dprev > 0.0 &&
                           dstep <= S.btol * fabs(S.energy) * (1.0 - fmin(fmax(dstep / S.dprev, 0.0), 0.99))) {
                    S.converged = 1;
                    S.done = 1;
                } else if (iter >= S.maxit) {
                    S.done = 1;
                }
                S.dprev = dstep;
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
        if (!own[j]) continue;
        const int idx = threadIdx.x + j * NT;
        gst(gx + idx, mk<T>(xr[j], xi[j]));
        gst(gr + idx, mk<T>(rr_[j], ri[j]));
        gst(gp + idx, mk<T>(pr[j], pi_[j]));
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        *a.st = S;
        if (a.mirror != nullptr) *a.mirror = S;
    }
}

// ---- best-iterate checkpoints of the FP32-iteration form ----
// Every CG iterate is admissible, so its exact energy is a guaranteed bound
// (Sec. 6.4); with FP32 iterates the recursively updated residual and the
// iterate drift apart once rounding dominates, and the energy of later
// iterates rises again.  A checkpoint measures the exact energy of the
// current iterate x: with b = -G A_M E the right-hand side and K the operator,
// (A_M (E + x), E + x) = (A_M E, E) - 2 (b, x) + (K x, x).

// Partials of (b, x) over the update grid (half-spectrum weights).
template <typename T>
__global__ __launch_bounds__(kThreads) void ckpt_dot_kernel(UpdArgs a, const Vt<T> *b, double *part, int final) {
    const CgStatus *st = a.st;
    if (st->done && !final) return;
    const Vt<T> *x = reinterpret_cast<const Vt<T> *>(a.x);
    double acc = 0.0;
    const long total = a.n_per_comp * a.nc;
    for (long idx = blockIdx.x * (long)kThreads + threadIdx.x; idx < total; idx += (long)a.nblocks * kThreads) {
        const long c = idx / a.n_per_comp;
        const long i = idx - c * a.n_per_comp;
        const long off = c * a.cs + i;
        const Vt<T> bv = b[off], xv = x[off];
        const double w = (i % a.Nh) == 0 ? 1.0 : 2.0;
        acc += w * ((double)bv.x * xv.x + (double)bv.y * xv.y);
    }
    const double s = block_sum(acc);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// The energy of x against the best one; sets the copy / restore flags.
__global__ __launch_bounds__(kThreads) void ckpt_decide_kernel(CgStatus *st, const double *part_xkx, int n_xkx,
                                                               const double *part_bx, int n_bx, int window,
                                                               int final) {
    const bool skip = final ? (st->converged || st->breakdown) : st->done;
    if (skip) {
        // a stalled solve keeps its restore mark (the copy is then repeated, with
        // the same result): solves that run together go on with their periodic
        // checkpoints until the last of them is done
        if (threadIdx.x == 0) {
            st->ck_copy = 0;
            if (final) st->ck_restore = 0;
        }
        return;
    }
    const double xkx = sum_fixed(part_xkx, n_xkx);
    const double bx = sum_fixed(part_bx, n_bx);
    if (threadIdx.x != 0) return;
    const double e = st->eAE - 2.0 * bx + xkx;
    st->ck_copy = 0;
    st->ck_restore = 0;
    if (final) {
        // keep the current iterate unless the kept copy is better
        if (!(e <= st->ebest)) st->ck_restore = 1;
        return;
    }
    if (isfinite(e) && e < st->ebest) {
        st->ebest = e;
        st->best_it = st->iter;
        st->ck_copy = 1;
        return;
    }
    // a rise far beyond the rounding of the FP32 operator (~1e-7 of the
    // energy), or no gain while the residual has made no new minimum for a
    // whole window: the iteration has stalled
    const bool rise = !isfinite(e) || e > st->ebest + 1e-5 * fabs(st->ebest);
    const bool stall = st->iter - st->rrmin_it >= window;
    if (rise || stall) {
        st->stagnated = 1;
        st->done = 1;
        st->ck_restore = 1;
    }
}

// Copy x into xbest or back, as the checkpoint decided.
template <typename T>
__global__ __launch_bounds__(kThreads) void ckpt_copy_kernel(UpdArgs a, Vt<T> *xbest) {
    const CgStatus *st = a.st;
    const int cp = st->ck_copy, rs = st->ck_restore;
    if (!cp && !rs) return;
    Vt<T> *x = reinterpret_cast<Vt<T> *>(a.x);
    const long total = a.n_per_comp * a.nc;
    for (long idx = blockIdx.x * (long)kThreads + threadIdx.x; idx < total; idx += (long)a.nblocks * kThreads) {
        const long c = idx / a.n_per_comp;
        const long off = c * a.cs + (idx - c * a.n_per_comp);
        if (cp)
            xbest[off] = x[off];
        else
            x[off] = xbest[off];
    }
}

__global__ void copy_words_kernel(unsigned int *dst, const unsigned int *src, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

// ---- matrix voxel images (eq. gridcomp with C^p in R^{d x d}) ----
// Determinant and inverse of a symmetric 2 x 2 or 3 x 3 matrix by cofactors.
__device__ __forceinline__ double sym_det(const double *m, int d) {
    if (d == 2) return m[0] * m[3] - m[1] * m[2];
    return m[0] * (m[4] * m[8] - m[5] * m[7]) - m[1] * (m[3] * m[8] - m[5] * m[6]) +
           m[2] * (m[3] * m[7] - m[4] * m[6]);
}

__device__ __forceinline__ void sym_inverse(const double *m, int d, double *out) {
    const double det = sym_det(m, d);
    if (d == 2) {
        out[0] = m[3] / det;
        out[1] = -m[1] / det;
        out[2] = -m[2] / det;
        out[3] = m[0] / det;
        return;
    }
    out[0] = (m[4] * m[8] - m[5] * m[7]) / det;
    out[1] = (m[2] * m[7] - m[1] * m[8]) / det;
    out[2] = (m[1] * m[5] - m[2] * m[4]) / det;
    out[3] = (m[5] * m[6] - m[3] * m[8]) / det;
    out[4] = (m[0] * m[8] - m[2] * m[6]) / det;
    out[5] = (m[2] * m[3] - m[0] * m[5]) / det;
    out[6] = (m[3] * m[7] - m[4] * m[6]) / det;
    out[7] = (m[1] * m[6] - m[0] * m[7]) / det;
    out[8] = (m[0] * m[4] - m[1] * m[3]) / det;
}

// A voxel matrix is accepted when finite, symmetric (to 1e-12 of its entries)
// and positive definite (leading principal minors > 0, Sylvester).
__global__ __launch_bounds__(kThreads) void tensor_check_kernel(const double *img, long n, int d, double *part) {
    double bad = 0.0;
    const int dd = d * d;
    for (long i = blockIdx.x * (long)kThreads + threadIdx.x; i < n; i += (long)gridDim.x * kThreads) {
        double m[9];
        bool ok = true;
        for (int k = 0; k < dd; ++k) {
            m[k] = img[i * dd + k];
            ok = ok && isfinite(m[k]);
        }
        for (int r = 0; r < d && ok; ++r)
            for (int c = r + 1; c < d; ++c)
                if (fabs(m[r * d + c] - m[c * d + r]) > 1e-12 * (fabs(m[r * d + c]) + fabs(m[c * d + r]))) ok = false;
        if (ok) {
            const double m1 = m[0];
            const double m2 = m[0] * m[d + 1] - m[1] * m[d];
            ok = m1 > 0.0 && m2 > 0.0 && (d == 2 || sym_det(m, d) > 0.0);
        }
        bad += ok ? 0.0 : 1.0;
    }
    const double s = block_sum(bad);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

__global__ __launch_bounds__(kThreads) void tensor_component_kernel(const double *img, long n, int d, int a, int b,
                                                                    int invert, double *out) {
    const int dd = d * d;
    for (long i = blockIdx.x * (long)kThreads + threadIdx.x; i < n; i += (long)gridDim.x * kThreads) {
        if (!invert) {
            out[i] = 0.5 * (img[i * dd + a * d + b] + img[i * dd + b * d + a]);
            continue;
        }
        double m[9], inv[9];
        for (int k = 0; k < dd; ++k) m[k] = img[i * dd + k];
        sym_inverse(m, d, inv);
        out[i] = 0.5 * (inv[a * d + b] + inv[b * d + a]);
    }
}

// Device-side validation of a voxel image: per work-group min, max and the
// number of entries that are not positive finite (part[3 b + 0..2]).
__global__ __launch_bounds__(kThreads) void image_stats_kernel(const double *img, long n, double *part) {
    double mn = INFINITY, mx = -INFINITY, bad = 0.0;
    for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
        const double v = img[i];
        if (!(v > 0.0) || !isfinite(v)) {
            bad += 1.0;
        } else {
            mn = fmin(mn, v);
            mx = fmax(mx, v);
        }
    }
    __shared__ double smn[kThreads], smx[kThreads], sbd[kThreads];
    smn[threadIdx.x] = mn;
    smx[threadIdx.x] = mx;
    sbd[threadIdx.x] = bad;
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            smn[threadIdx.x] = fmin(smn[threadIdx.x], smn[threadIdx.x + w]);
            smx[threadIdx.x] = fmax(smx[threadIdx.x], smx[threadIdx.x + w]);
            sbd[threadIdx.x] += sbd[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[3 * blockIdx.x + 0] = smn[0];
        part[3 * blockIdx.x + 1] = smx[0];
        part[3 * blockIdx.x + 2] = sbd[0];
    }
}

// out[0..3] = min, max, #invalid, #entries equal to neither min nor max.
__global__ __launch_bounds__(kThreads) void image_stats_reduce(const double *part, int nb, double *out) {
    if (threadIdx.x == 0) {
        double mn = INFINITY, mx = -INFINITY, bad = 0.0;
        for (int b = 0; b < nb; ++b) {
            mn = fmin(mn, part[3 * b]);
            mx = fmax(mx, part[3 * b + 1]);
            bad += part[3 * b + 2];
        }
        out[0] = mn;
        out[1] = mx;
        out[2] = bad;
    }
}

__global__ __launch_bounds__(kThreads) void image_other_kernel(const double *img, long n, const double *mm,
                                                               double *part) {
    const double mn = mm[0], mx = mm[1];
    double cnt = 0.0;
    for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
        const double v = img[i];
        if (v != mn && v != mx) cnt += 1.0;
    }
    const double s = block_sum(cnt);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
// ---------------------------------------------------------------------------
// ---------------------------------------------------------------------------
template <int... I>
static void fill_parts(FastKernels *t, std::integer_sequence<int, I...>) {
    (fill_fast<I>(t), ...);
}
const FastKernels &fast_kernels(int fi) {
    struct Table {
        FastKernels k[kNumFast];
        Table() { fill_parts(k, std::make_integer_sequence<int, kFastParts>()); }
    };
    static const Table t;
    return t.k[fi];
}

// The table entry of a pass that configure_pencil / configure_row gave a
// specialised kernel: pencils 1 (a length of kFastSched), 2 (Bluestein), 3 and 4
// (the same for the two components of 3D gradient fields); rows
// 1 (any material; energy Gram), 2 (isotropic, single transforms), 3
// (isotropic, whole row pairs), 4 and 5 (Bluestein: whole row pairs, single), 6
// (isotropic, planes).
static const FastKernels::Pencil &fast_pencil(const PencilArgs &a, bool fp64) {
    const FastKernels &k = fast_kernels(fast_index(a.f.L));
    switch (a.fast) {
        case 1: return k.pencil[fp64][a.d - 2];
        case 2: return k.blue_pencil[fp64][a.d - 2];
        case 3: return k.pencil2[fp64];
        default: return k.blue_pencil2[fp64];
    }
}
static const FastKernels::Row &fast_row(const RowArgs &a, bool fp64) {
    const FastKernels &k = fast_kernels(fast_index(a.f.L));
    if (a.mode == ROW_GRAM) return k.gram[a.d - 2];
    switch (a.fast) {
        case 1: return k.row[fp64][a.d - 2];
        case 2: return k.iso[fp64][a.d - 2];
        case 3: return k.pairs[fp64][a.d - 2];
        case 6: return k.plane[fp64];
        default: return k.blue_row[fp64][a.d - 2];
    }
}

size_t pencil_lds_bytes(const PencilArgs &a, bool fp64) {
    const size_t es = fp64 ? 16 : 8;
    if (a.fast) return fast_pencil(a, fp64).lds;
    int lacc = 0;
    if (a.pro == PRO_EXPAND) lacc = a.nc * a.L_in;
    if (a.epi == EPI_PROJECT) lacc = a.nc * a.L_out;
    return es * ((size_t)2 * a.f.L * std::max(a.cb, 1) * a.B + (size_t)lacc * a.B + (size_t)std::max(a.twl, 0));
}

size_t row_lds_bytes(const RowArgs &a, bool fp64) {
    const size_t es = fp64 ? 16 : 8;
    if (a.fast) {
        return fast_row(a, fp64).lds;
    }
    const int nz = row_zbufs(a);
    return es * (size_t)(a.zbatch ? 2 * nz : nz + 1) * a.RP * a.f.L;
}

int pencil_grid_x(const PencilArgs &a) { return a.B > 0 ? (a.nb + a.B - 1) / a.B : 0; }
int row_grid(const RowArgs &a) {
    if (a.RP < 1) return 0;
    if (a.fast == 6) return a.nrows;
    if (a.mode == ROW_GRAM && a.gpack && !a.fast) return (a.nrows + a.RP - 1) / a.RP;
    const int pairs = (a.nrows + 1) / 2;
    if (a.fast == 3 || a.fast == 4) return (pairs + a.RP / a.d - 1) / (a.RP / a.d);
    return a.fast == 2 || a.fast == 5 ? (a.d * pairs + a.RP - 1) / a.RP : (pairs + a.RP - 1) / a.RP;
}

// Index in kFastSched of the transform (Bluestein: convolution) length of f
// when its stages are that schedule, else -1.
static int fast_of(const FftDesc &f) {
    const int fi = fast_index(f.L);
    if (fi < 0 || f.nst != kFastSched[fi].nst) return -1;
    for (int s = 0; s < f.nst; ++s)
        if (f.radix[s] != kFastSched[fi].r[s]) return -1;
    return fi;
}

bool fast_pencils(const FftDesc &f, bool fp64) {
    const int fi = fast_of(f);
    if (fi < 0) return false;
    const FastKernels &k = fast_kernels(fi);
    return f.blue ? k.blue_pencil[fp64][1].fn && k.blue_pencil2[fp64].fn
                  : k.pencil[fp64][1].fn && k.pencil2[fp64].fn;
}

void configure_pencil(PencilArgs &a, bool fp64) {
    const int fi = fast_of(a.f);
    const bool two = a.d == 3 && a.ncomp == 2;
    if (fi >= 0 && a.nsol == 1 && (a.ncomp == a.d || two) && a.epi != EPI_WINDOW && (a.d == 2 || a.d == 3) &&
        a.L_in <= a.f.n && a.L_out <= a.f.n) {
        a.fast = (a.f.blue ? 2 : 1) + (two ? 2 : 0);
        if (fast_pencil(a, fp64).fn) {
            a.B = fast_pencil(a, fp64).B;
            return;
        }
    }
    a.fast = 0;
    a.cb = 1;
    a.twl = 0;
    a.B = fp64 ? 8 : 16;
    while (a.B > 1 && pencil_lds_bytes(a, fp64) > kGenericLds) a.B /= 2;
    fit_pencil_components(a, fp64);
}

void fit_pencil_components(PencilArgs &a, bool fp64) {
    a.twl = 0;
    a.cb = std::max(a.ncomp, 1);
    while (a.cb > 1 && pencil_lds_bytes(a, fp64) > kGenericLds) --a.cb;
    // then the table in LDS, if it fits too: the stage twiddles (L - 1
    // entries), for Bluestein followed by the chirp (n) and the filter (L)
    if (a.f.nst < 1) return;
    a.twl = a.f.blue ? a.f.hoff + a.f.L - a.f.twoff[0] : a.f.L - 1;
    if (a.twl < 1 || pencil_lds_bytes(a, fp64) > kGenericLds) a.twl = 0;
}

bool plane_fits(const FftDesc &f, int L2, int nh, bool fp64) {
    const int fi = fast_of(f);
    if (fi < 0 || f.blue) return false;
    const FastKernels::Row &e = fast_kernels(fi).plane[fp64];
    return e.fn && nh <= e.nh_max && 2 * L2 <= f.n + 1;
}

void configure_row(RowArgs &r, bool fp64) {
    if (r.L2 > 0) {  // plane_fits
        r.fast = 6;
        r.RP = 1;
        return;
    }
    const int fi = fast_of(r.f);
    if (fi >= 0 && (r.d == 2 || r.d == 3)) {
        const FastKernels &k = fast_kernels(fi);
        const bool oper = r.mode == ROW_OPER && r.ncomp == r.d;
        auto take = [&](const FastKernels::Row &e, int fast) {
            if (!e.fn || r.Nh_row > e.nh_max) return false;
            r.fast = fast;
            r.RP = e.RP;
            return true;
        };
        if (r.f.blue) {
            const FastKernels::Row &e = k.blue_row[fp64][r.d - 2];
            if (oper && r.iso && take(e, e.RP > 1 ? 4 : 5)) return;
        } else {
            if (oper && r.iso && take(k.pairs[fp64][r.d - 2], 3)) return;
            if (oper && r.iso && take(k.iso[fp64][r.d - 2], 2)) return;
            if ((oper || (r.mode == ROW_RHS && r.ncomp == r.d)) && take(k.row[fp64][r.d - 2], 1)) return;
            if (fp64 && r.mode == ROW_GRAM && r.ncomp == r.d * r.d && take(k.gram[r.d - 2], 1)) return;
        }
    }
    r.fast = 0;
    r.zbatch = 0;
    r.gpack = 0;
    r.RP = 1;
    if (r.mode == ROW_GRAM && row_lds_bytes(r, fp64) > kGenericLds) r.gpack = 1;  // long rows: two components of one row per transform
    r.RP = 8;
    while (r.RP > 1 && row_lds_bytes(r, fp64) > kGenericLds) r.RP /= 2;
    fit_row_batch(r, fp64);
}

void fit_row_batch(RowArgs &r, bool fp64) {
    r.zbatch = 0;
    if (r.fast || r.gpack || row_zbufs(r) < 2) return;
    r.zbatch = 1;
    if (row_lds_bytes(r, fp64) > kGenericLds) r.zbatch = 0;
}

// Whether the generic kernels take f in their form with radices 11 and 13.  In
// one kernel with all eight radices the row passes kept their arguments in
// scratch memory (620 bytes, one wave per SIMD against three): the energies of
// 3D GaNi fields of order 225 on 525^3 took 141 ms instead of 40.
static bool has_13(const FftDesc &f) {
    for (int st = 0; st < f.nst; ++st)
        if (f.radix[st] == 11 || f.radix[st] == 13) return true;
    return false;
}

hipError_t launch_pencil(const PencilArgs &a, int nouter, bool fp64, hipStream_t s) {
    if (a.B < 1 || nouter < 1 || a.fast) return hipErrorInvalidValue;
    dim3 grid(pencil_grid_x(a), nouter);
    const size_t lds = pencil_lds_bytes(a, fp64);
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(kThreads), lds, s, a); };
    if (has_13(a.f))
        fp64 ? go(pencil_kernel<double, true>) : go(pencil_kernel<float, true>);
    else
        fp64 ? go(pencil_kernel<double, false>) : go(pencil_kernel<float, false>);
    return hipGetLastError();
}

hipError_t launch_row(const RowArgs &a, bool fp64, hipStream_t s) {
    if (a.RP < 1 || a.fast) return hipErrorInvalidValue;
    const size_t lds = row_lds_bytes(a, fp64);
    if (a.d != 2 && a.d != 3) return hipErrorInvalidValue;
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(row_grid(a)), dim3(kThreads), lds, s, a); };
    if (has_13(a.f)) {
        if (a.d == 3)
            fp64 ? go(row_kernel<double, 3, true>) : go(row_kernel<float, 3, true>);
        else
            fp64 ? go(row_kernel<double, 2, true>) : go(row_kernel<float, 2, true>);
    } else {
        if (a.d == 3)
            fp64 ? go(row_kernel<double, 3, false>) : go(row_kernel<float, 3, false>);
        else
            fp64 ? go(row_kernel<double, 2, false>) : go(row_kernel<float, 2, false>);
    }
    return hipGetLastError();
}

// Index of the compile-time grid of the single-work-group solver, or -1.
static int solo_fast(int m) {
    const int fi = fast_index(m);
    return fi == 0 || fi == 1 ? fi : -1;
}
static size_t solo_lds(int M0, int M1, bool fp64) {
    return fp64 ? solo_lds_bytes_t<double>(M0, M1) : solo_lds_bytes_t<float>(M0, M1);
}
constexpr size_t kSoloLds = 160 * 1024 - 1024;

// Threads of the run-time-length form: few on small grids, then whatever the
// registers of the in-place stages (solo_per) and of the CG vectors
// (solo_cpt) need; 0 if the grid does not fit.
// A serial chain of stages and barriers bounds the kernel, so threads without
// work only cost barriers.  2D order 11 (21 x 21), FP64: 29 us per iteration in five
// launches of single passes -> 4.4 us here.
static int solo_threads(const SoloArgs &a, bool fp64) {
    const long pts = (long)a.M0 * a.M1;
    for (int nt = pts <= 1500 ? 256 : pts <= 4000 ? 512 : 1024; nt <= 1024; nt *= 2) {
        bool ok = (long)a.N0 * a.Nh <= (long)nt * solo_cpt(-1, -1, nt);
        for (int x = 0; x < 2; ++x)
            for (int s = 0; s < a.nst[x]; ++s) {
                const SoloStage &g = a.stg[x][s];
                ok = ok && (long)g.TQ * (x == 0 ? 2 * a.Nh - 1 : a.M0) <= (long)nt * solo_per(g.R, fp64);
            }
        if (ok) return nt;
    }
    return 0;
}

bool solo_fits(SoloArgs &a, const FftDesc *f, bool fp64) {
    if (f[0].blue || f[1].blue || solo_lds(a.M0, a.M1, fp64) > kSoloLds) return false;
    if (solo_fast(a.M0) >= 0 && solo_fast(a.M1) >= 0) return true;
    auto mult = [](int d) { return d == 1 ? 0u : (unsigned)((1ull << 32) / (unsigned)d) + 1u; };
    for (int x = 0; x < 2; ++x) {
        if (f[x].nst > kSoloStages) return false;
        a.nst[x] = f[x].nst;
        int p = 1;
        for (int s = 0; s < f[x].nst; ++s) {
            const int r = f[x].radix[s];
            if (r != 3 && r != 5 && r != 7 && r != 9 && r != 15 && r != 25) return false;
            a.stg[x][s] = {r, p, f[x].n / r, f[x].twoff[s] - f[x].twoff[0], mult(f[x].n / r), mult(p)};
            p *= r;
        }
    }
    a.mNh = mult(a.Nh);
    a.mNA = mult(2 * a.Nh - 1);
    return solo_threads(a, fp64) > 0;
}

template <typename T, int FI0, int FI1>
void launch_solo_t(const SoloArgs *args, int np, int niter, const Disp &s) {
    constexpr size_t lds = solo_lds_bytes_t<T>(kFastSched[FI0].n, kFastSched[FI1].n);
    if constexpr (lds <= kSoloLds)
        dispatch((solo2d_kernel<T, FI0, FI1, kSoloNT>), dim3(np), dim3(kSoloNT), lds, s, args, niter);
}

template <typename T>
void launch_solo_d(const SoloArgs &proto, const SoloArgs *args, int np, int niter, const Disp &s) {
    const int f0 = solo_fast(proto.M0), f1 = solo_fast(proto.M1);
    if (f0 < 0 || f1 < 0) {
        const size_t lds = solo_lds_bytes_t<T>(proto.M0, proto.M1);
        const int nt = solo_threads(proto, sizeof(T) == 8);
        if (nt == 256) dispatch((solo2d_kernel<T, -1, -1, 256>), dim3(np), dim3(256), lds, s, args, niter);
        if (nt == 512) dispatch((solo2d_kernel<T, -1, -1, 512>), dim3(np), dim3(512), lds, s, args, niter);
        if (nt == 1024) dispatch((solo2d_kernel<T, -1, -1, 1024>), dim3(np), dim3(1024), lds, s, args, niter);
        return;
    }
    if (f0 == 0 && f1 == 0) launch_solo_t<T, 0, 0>(args, np, niter, s);
    if (f0 == 0 && f1 == 1) launch_solo_t<T, 0, 1>(args, np, niter, s);
    if (f0 == 1 && f1 == 0) launch_solo_t<T, 1, 0>(args, np, niter, s);
    if (f0 == 1 && f1 == 1) launch_solo_t<T, 1, 1>(args, np, niter, s);
}

hipError_t launch_solo(const SoloArgs &proto, const SoloArgs *args, int np, int niter, bool fp64, hipStream_t st,
                       LaunchEv ev) {
    if (np < 1 || niter < 1 || solo_lds(proto.M0, proto.M1, fp64) > kSoloLds) return hipErrorInvalidValue;
    if ((solo_fast(proto.M0) < 0 || solo_fast(proto.M1) < 0) && solo_threads(proto, fp64) == 0)
        return hipErrorInvalidValue;
    const Disp s(st, ev);
    if (fp64)
        launch_solo_d<double>(proto, args, np, niter, s);
    else
        launch_solo_d<float>(proto, args, np, niter, s);
    return hipGetLastError();
}

int pencil_grid(const PencilArgs &a, int nouter) { return pencil_grid_x(a) * nouter; }
int update_blocks(long n) { return (int)std::max<long>(1, (n + (long)kThreads * kUpdPer - 1) / ((long)kThreads * kUpdPer)); }

hipError_t launch_pencil_multi(const PencilArgs &proto, const PencilArgs *args, const int *woff, int np, int total,
                               bool fp64, hipStream_t st, LaunchEv ev) {
    if (!proto.fast || fast_index(proto.f.L) < 0 || np < 1 || total < 1) return hipErrorInvalidValue;
    const FastKernels::Pencil &e = fast_pencil(proto, fp64);
    if (!e.fn) return hipErrorInvalidValue;
    e.fn(args, woff, np, total, st, ev);
    return hipGetLastError();
}

hipError_t launch_row_multi(const RowArgs &proto, const RowArgs *args, const int *woff, int np, int total, bool fp64,
                            hipStream_t st, LaunchEv ev) {
    if (!proto.fast || fast_index(proto.f.L) < 0 || np < 1 || total < 1) return hipErrorInvalidValue;
    const FastKernels::Row &e = fast_row(proto, fp64);
    if (!e.fn || (proto.mode == ROW_GRAM && !fp64) || (proto.fast > 1 && proto.mode != ROW_OPER))
        return hipErrorInvalidValue;
    e.fn(args, woff, np, total, st, ev);
    return hipGetLastError();
}

hipError_t launch_cg_check_multi(const CgItem *items, int np, hipStream_t st, LaunchEv ev) {
    dispatch(cg_check_multi_kernel, dim3(np), dim3(kThreads), 0, Disp(st, ev), items);
    return hipGetLastError();
}

hipError_t launch_cg_update_multi(const UpdArgs *ua, const int *woff, int np, int total, bool fp64, hipStream_t st,
                                  LaunchEv ev) {
    const Disp s(st, ev);
    if (fp64)
        dispatch(cg_update_multi_kernel<double>, dim3(total), dim3(kThreads), 0, s, ua, woff, np);
    else
        dispatch(cg_update_multi_kernel<float>, dim3(total), dim3(kThreads), 0, s, ua, woff, np);
    return hipGetLastError();
}

hipError_t launch_cg_checkpoint(const UpdArgs &u, const void *b, void *xbest, const double *part_xkx, int n_xkx,
                                double *part_bx, int window, int final, bool fp64, hipStream_t s) {
    if (fp64)
        hipLaunchKernelGGL(ckpt_dot_kernel<double>, dim3(u.nblocks), dim3(kThreads), 0, s, u,
                           reinterpret_cast<const double2 *>(b), part_bx, final);
    else
        hipLaunchKernelGGL(ckpt_dot_kernel<float>, dim3(u.nblocks), dim3(kThreads), 0, s, u,
                           reinterpret_cast<const float2 *>(b), part_bx, final);
    hipLaunchKernelGGL(ckpt_decide_kernel, dim3(1), dim3(kThreads), 0, s, u.st, part_xkx, n_xkx, part_bx, u.nblocks,
                       window, final);
    if (fp64)
        hipLaunchKernelGGL(ckpt_copy_kernel<double>, dim3(u.nblocks), dim3(kThreads), 0, s, u,
                           reinterpret_cast<double2 *>(xbest));
    else
        hipLaunchKernelGGL(ckpt_copy_kernel<float>, dim3(u.nblocks), dim3(kThreads), 0, s, u,
                           reinterpret_cast<float2 *>(xbest));
    return hipGetLastError();
}

hipError_t launch_tensor_check(const double *img, long n, int d, double *part, int *nparts, hipStream_t s) {
    const int blocks = (int)std::max<long>(1, std::min<long>((n + kThreads - 1) / kThreads, 1024));
    *nparts = blocks;
    hipLaunchKernelGGL(tensor_check_kernel, dim3(blocks), dim3(kThreads), 0, s, img, n, d, part);
    return hipGetLastError();
}

hipError_t launch_tensor_component(const double *img, long n, int d, int a, int b, int invert, double *out,
                                   hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int blocks = (int)std::min<long>((n + kThreads - 1) / kThreads, 4096);
    hipLaunchKernelGGL(tensor_component_kernel, dim3(blocks), dim3(kThreads), 0, s, img, n, d, a, b, invert, out);
    return hipGetLastError();
}

hipError_t launch_copy_vec(void *dst, const void *src, size_t bytes, hipStream_t s) {
    if (bytes % 4) return hipErrorInvalidValue;
    const size_t n = bytes / 4;
    if (n == 0) return hipSuccess;
    const int blocks = (int)std::min<size_t>((n + kThreads - 1) / kThreads, 4096);
    hipLaunchKernelGGL(copy_words_kernel, dim3(blocks), dim3(kThreads), 0, s, reinterpret_cast<unsigned int *>(dst),
                       reinterpret_cast<const unsigned int *>(src), n);
    return hipGetLastError();
}

hipError_t launch_cg_init(const InitArgs &a, hipStream_t s) {
    hipLaunchKernelGGL(cg_init_kernel, dim3(1), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_cg_init_multi(const InitArgs *args, int np, hipStream_t s) {
    hipLaunchKernelGGL(cg_init_multi_kernel, dim3(np), dim3(kThreads), 0, s, args);
    return hipGetLastError();
}

hipError_t launch_vec_ops(const VecOps &ops, hipStream_t s) {
    size_t most = 0;
    for (int i = 0; i < ops.n; ++i) most = std::max<size_t>(most, ops.op[i].words);
    if (most == 0) return hipSuccess;
    const int nb = (int)std::min<size_t>((most + kThreads - 1) / kThreads, 2048);
    hipLaunchKernelGGL(vec_ops_kernel, dim3(nb, ops.n), dim3(kThreads), 0, s, ops);
    return hipGetLastError();
}

hipError_t launch_warm_residual(const UpdArgs &u, double *part_rr, double *part_bx, double *part_rx, bool fp64,
                                hipStream_t s) {
    if (fp64)
        hipLaunchKernelGGL(warm_residual_kernel<double>, dim3(u.nblocks), dim3(kThreads), 0, s, u, part_rr, part_bx,
                           part_rx);
    else
        hipLaunchKernelGGL(warm_residual_kernel<float>, dim3(u.nblocks), dim3(kThreads), 0, s, u, part_rr, part_bx,
                           part_rx);
    return hipGetLastError();
}

hipError_t launch_cg_init_warm(CgStatus *st, const double *part_rr, const double *part_bx, const double *part_rx,
                               int nparts, const double *scal, double mtot, double tol, double floor_rel, int maxit,
                               double btol, double *hist, hipStream_t s) {
    hipLaunchKernelGGL(cg_init_warm_kernel, dim3(1), dim3(kThreads), 0, s, st, part_rr, part_bx, part_rx, nparts,
                       scal, mtot, tol, floor_rel, maxit, btol, hist);
    return hipGetLastError();
}

hipError_t launch_sample_incl(double *g, int d, const int *M, const InclDev *inc, int n, double w0, hipStream_t s) {
    const int m0 = M[0], m1 = M[1], m2 = d == 3 ? M[2] : 1;
    const long total = (long)m0 * m1 * m2;
    const int blocks = (int)std::max<long>(1, std::min<long>(2048, (total + kThreads - 1) / kThreads));
    hipLaunchKernelGGL(sample_incl_kernel, dim3(blocks), dim3(kThreads), 0, s, g, d, m0, m1, m2, inc, n, w0);
    return hipGetLastError();
}

hipError_t launch_sample_voxel(double *g, const double *img, int d, const int *P, const int *M, int map, double vmax,
                               hipStream_t s) {
    const int m0 = M[0], m1 = M[1], m2 = d == 3 ? M[2] : 1;
    const int p0 = P[0], p1 = P[1], p2 = d == 3 ? P[2] : 1;
    const long total = (long)m0 * m1 * m2;
    const int blocks = (int)std::max<long>(1, std::min<long>(2048, (total + kThreads - 1) / kThreads));
    hipLaunchKernelGGL(sample_voxel_kernel, dim3(blocks), dim3(kThreads), 0, s, g, img, p0, p1, p2, m0, m1, m2, map,
                       vmax);
    return hipGetLastError();
}

hipError_t launch_envelope(double *upper, double *lower, int d, const int *P, const InclDev *inc, int n,
                           const double *ext, hipStream_t s) {
    const int p0 = P[0], p1 = P[1], p2 = d == 3 ? P[2] : 1;
    const long total = (long)p0 * p1 * p2;
    const int blocks = (int)std::max<long>(1, std::min<long>(2048, (total + kThreads - 1) / kThreads));
    hipLaunchKernelGGL(envelope_kernel, dim3(blocks), dim3(kThreads), 0, s, upper, lower, d, p0, p1, p2, inc, n, ext);
    return hipGetLastError();
}

hipError_t launch_fold_series(void *out, const void *coef, int d, const int *N, const int *L, int Lh,
                              const int *shift, hipStream_t s) {
    const int n0 = N[0], n1 = d == 3 ? N[1] : 1, n2 = N[d - 1];
    const long total = (d == 3 ? (long)n0 * n1 : (long)n0) * ((n2 + 1) / 2);
    const int blocks = (int)std::max<long>(1, std::min<long>(4096, (total + kThreads - 1) / kThreads));
    hipLaunchKernelGGL(fold_series_kernel, dim3(blocks), dim3(kThreads), 0, s, reinterpret_cast<double2 *>(out),
                       reinterpret_cast<const double2 *>(coef), d, n0, n1, n2, L[0], d == 3 ? L[1] : 1, Lh, shift[0],
                       d == 3 ? shift[1] : 0, shift[d - 1]);
    return hipGetLastError();
}

hipError_t launch_prolong(const void *src, bool src64, void *dst, bool dst64, int d, int nc, const int *Nf,
                          const int *Nc, hipStream_t s) {
    const int f1 = Nf[0], f2 = d == 3 ? Nf[1] : 1, f3h = (Nf[d - 1] + 1) / 2;
    const int c1 = Nc[0], c2 = d == 3 ? Nc[1] : 1, c3h = (Nc[d - 1] + 1) / 2;
    const long total = (long)f1 * f2 * f3h * nc;
    const int blocks = (int)std::max<long>(1, std::min<long>(1024, (total + kThreads - 1) / kThreads));
    if (src64 && dst64)
        hipLaunchKernelGGL((prolong_kernel<double, double>), dim3(blocks), dim3(kThreads), 0, s,
                           static_cast<const double2 *>(src), static_cast<double2 *>(dst), d, nc, f1, f2, f3h, c1, c2,
                           c3h);
    else if (src64)
        hipLaunchKernelGGL((prolong_kernel<double, float>), dim3(blocks), dim3(kThreads), 0, s,
                           static_cast<const double2 *>(src), static_cast<float2 *>(dst), d, nc, f1, f2, f3h, c1, c2,
                           c3h);
    else if (dst64)
        hipLaunchKernelGGL((prolong_kernel<float, double>), dim3(blocks), dim3(kThreads), 0, s,
                           static_cast<const float2 *>(src), static_cast<double2 *>(dst), d, nc, f1, f2, f3h, c1, c2,
                           c3h);
    else
        hipLaunchKernelGGL((prolong_kernel<float, float>), dim3(blocks), dim3(kThreads), 0, s,
                           static_cast<const float2 *>(src), static_cast<float2 *>(dst), d, nc, f1, f2, f3h, c1, c2,
                           c3h);
    return hipGetLastError();
}




hipError_t launch_fill_zero(void *p, size_t bytes, hipStream_t s) {
    const size_t nw = bytes / 4;
    if (nw == 0) return hipSuccess;
    const int nb = (int)std::min<size_t>((nw + kThreads - 1) / kThreads, 4096);
    hipLaunchKernelGGL(fill_zero_kernel, dim3(nb), dim3(kThreads), 0, s, (unsigned int *)p, nw);
    return hipGetLastError();
}

hipError_t launch_convert_f2d(double *dst, const float *src, size_t n, hipStream_t s) {
    const int nb = (int)std::min<size_t>((n + kThreads - 1) / kThreads, 4096);
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(f2d_kernel, dim3(nb), dim3(kThreads), 0, s, dst, src, n);
    return hipGetLastError();
}

hipError_t launch_convert_d2f(float *dst, const double *src, size_t n, hipStream_t s) {
    const int nb = (int)std::min<size_t>((n + kThreads - 1) / kThreads, 4096);
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(d2f_kernel, dim3(nb), dim3(kThreads), 0, s, dst, src, n);
    return hipGetLastError();
}

hipError_t launch_sum_partials(double *out, const double *part, int nparts, int nvals, hipStream_t s) {
    if (nvals < 1) return hipSuccess;
    hipLaunchKernelGGL(sum_partials_kernel, dim3(nvals), dim3(kThreads), 0, s, out, part, nparts, nvals);
    return hipGetLastError();
}

hipError_t launch_image_stats(const double *img, long n, double *part, double *out, hipStream_t s) {
    const int nb = 256;  // 3 * nb partials fit the plan's partial-sum region
    hipLaunchKernelGGL(image_stats_kernel, dim3(nb), dim3(kThreads), 0, s, img, n, part);
    hipLaunchKernelGGL(image_stats_reduce, dim3(1), dim3(kThreads), 0, s, part, nb, out);
    hipLaunchKernelGGL(image_other_kernel, dim3(nb), dim3(kThreads), 0, s, img, n, out, part);
    hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(kThreads), 0, s, out + 3, part, nb, 1);
    return hipGetLastError();
}

hipError_t launch_incl_coeff(void *out, int d, int L1, int L2, int Lh, const InclDev *incl, int n_incl,
                             double w0, hipStream_t s) {
    const long total = (d == 3 ? (long)L1 * L2 * Lh : (long)L1 * Lh);
    const int nb = (int)std::min<long>((total + kThreads - 1) / kThreads, 8192);
    hipLaunchKernelGGL(incl_coeff_kernel, dim3(nb), dim3(kThreads), 0, s, (double2 *)out, d, L1, L2, Lh, incl,
                       n_incl, w0);
    return hipGetLastError();
}

}  // namespace fftgal
