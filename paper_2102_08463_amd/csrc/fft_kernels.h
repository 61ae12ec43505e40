// Fine-grid FFT with the truncation, zero padding and correction factors of
// Sec. II-A step 3 and Sec. II-B step 1 inside its passes.
//
// One pass transforms every line of the grid along one dimension: a block
// loads C lines into registers, exchanges them between radix stages through
// LDS (Stockham order, so nothing is bit-reversed) and stores them.  Type 1
// keeps N of the n outputs of each dimension and scales them in its last
// pass; type 2 reads the N inputs, scaled, in its first pass and zeros
// elsewhere.  A dimension that has been cut to N (or not yet been padded to
// n) is not transformed outside those N lines, so in 2D at sigma = 2 a
// transform moves 1 read + 1/2 write + 1/2 read + 1/4 write of the grid
// against 2 reads + 2 writes for a full FFT and its own pass for the factors.
//
// What bounds it: HBM / Infinity Cache traffic in 64 to 128 B pieces; the
// radix stages need a few FMAs per byte and two LDS exchanges (n up to 4096).
// Column tiles are numbered so that each XCD takes neighbouring ones, whose
// lines meet in its L2.
#pragma once
#include "internal.h"

namespace mn {
namespace fft {

template <typename T> struct Cplx;
template <> struct Cplx<float> { using type = float2; };
template <> struct Cplx<double> { using type = double2; };

// ---- radix butterflies ------------------------------------------------------
constexpr double kPi = 3.141592653589793238462643383;

// cos and sin of x in [0, pi/4] by Taylor series (error below 1e-17).
constexpr double cos_small(double x)
{
    double t = 1.0, s = 1.0;
    for (int k = 1; k < 14; ++k) {
        t *= -x * x / ((2 * k - 1) * (2 * k));
        s += t;
    }
    return s;
}
constexpr double sin_small(double x)
{
    double t = x, s = x;
    for (int k = 1; k < 14; ++k) {
        t *= -x * x / ((2 * k) * (2 * k + 1));
        s += t;
    }
    return s;
}
// cos(2 pi k / R) with the angle folded into the first octant exactly.
constexpr double cos2pi(int k, int R)
{
    k %= R;
    if (k < 0) k += R;
    if (2 * k > R) k = R - k;               // cos(2 pi - a) = cos a
    double sg = 1.0;
    int num = k;                            // angle = 2 pi num / R, num <= R / 2
    if (4 * num > R) {                      // cos(pi - a) = -cos a
        sg = -1.0;
        return 8 * (R - 2 * num) <= 2 * R
                   ? sg * cos_small(kPi * (R - 2 * num) / R)
                   : sg * sin_small(kPi * (4 * num - R) / (2.0 * R));
    }
    return 8 * num <= R ? cos_small(2 * kPi * num / R) : sin_small(kPi * (R - 4 * num) / (2.0 * R));
}
constexpr double sin2pi(int k, int R) { return cos2pi(4 * k - R, 4 * R); }

// v *= exp(-2 pi i K / R)
template <int K, int R, typename C>
__device__ __forceinline__ void rot(C &v)
{
    if constexpr (K % R == 0) {
        return;
    } else if constexpr (4 * (K % R) == R) {
        const auto t = v.x;
        v.x = v.y;
        v.y = -t;
    } else if constexpr (2 * (K % R) == R) {
        v.x = -v.x;
        v.y = -v.y;
    } else if constexpr (4 * (K % R) == 3 * R) {
        const auto t = v.x;
        v.x = -v.y;
        v.y = t;
    } else {
        using T = decltype(v.x + v.x);
        constexpr T c = (T)cos2pi(K, R), s = (T)sin2pi(K, R);
        const T a = v.x * c + v.y * s;
        v.y = v.y * c - v.x * s;
        v.x = a;
    }
}

// In-place forward DFT of x[0], x[S], ..., x[(R - 1) S].
template <int R, typename C> struct Dft;

template <typename C> struct Dft<2, C> {
    template <int S> static __device__ __forceinline__ void go(C *x)
    {
        const C a = x[0], b = x[S];
        x[0].x = a.x + b.x; x[0].y = a.y + b.y;
        x[S].x = a.x - b.x; x[S].y = a.y - b.y;
    }
};
template <typename C> struct Dft<3, C> {
    template <int S> static __device__ __forceinline__ void go(C *x)
    {
        using T = decltype(x[0].x + x[0].x);
        constexpr T s3 = (T)sin2pi(1, 3);
        const C a = x[0];
        const T sx = x[S].x + x[2 * S].x, sy = x[S].y + x[2 * S].y;
        const T dx = (x[S].x - x[2 * S].x) * s3, dy = (x[S].y - x[2 * S].y) * s3;
        const T mx = a.x - (T)0.5 * sx, my = a.y - (T)0.5 * sy;
        x[0].x = a.x + sx; x[0].y = a.y + sy;
        x[S].x = mx + dy; x[S].y = my - dx;
        x[2 * S].x = mx - dy; x[2 * S].y = my + dx;
    }
};
template <typename C> struct Dft<4, C> {
    template <int S> static __device__ __forceinline__ void go(C *x)
    {
        const C a = x[0], b = x[S], c = x[2 * S], d = x[3 * S];
        const C e = {a.x + c.x, a.y + c.y}, f = {a.x - c.x, a.y - c.y};
        const C g = {b.x + d.x, b.y + d.y}, h = {b.x - d.x, b.y - d.y};
        x[0].x = e.x + g.x; x[0].y = e.y + g.y;
        x[2 * S].x = e.x - g.x; x[2 * S].y = e.y - g.y;
        x[S].x = f.x + h.y; x[S].y = f.y - h.x;
        x[3 * S].x = f.x - h.y; x[3 * S].y = f.y + h.x;
    }
};
template <typename C> struct Dft<5, C> {
    template <int S> static __device__ __forceinline__ void go(C *x)
    {
        using T = decltype(x[0].x + x[0].x);
        constexpr T c1 = (T)cos2pi(1, 5), c2 = (T)cos2pi(2, 5);
        constexpr T s1 = (T)sin2pi(1, 5), s2 = (T)sin2pi(2, 5);
        const C a = x[0];
        const C p = {x[S].x + x[4 * S].x, x[S].y + x[4 * S].y};
        const C q = {x[2 * S].x + x[3 * S].x, x[2 * S].y + x[3 * S].y};
        const C m = {x[S].x - x[4 * S].x, x[S].y - x[4 * S].y};
        const C r = {x[2 * S].x - x[3 * S].x, x[2 * S].y - x[3 * S].y};
        const C u = {a.x + c1 * p.x + c2 * q.x, a.y + c1 * p.y + c2 * q.y};
        const C v = {a.x + c2 * p.x + c1 * q.x, a.y + c2 * p.y + c1 * q.y};
        const C g = {s1 * m.x + s2 * r.x, s1 * m.y + s2 * r.y};
        const C h = {s2 * m.x - s1 * r.x, s2 * m.y - s1 * r.y};
        x[0].x = a.x + p.x + q.x; x[0].y = a.y + p.y + q.y;
        x[S].x = u.x + g.y; x[S].y = u.y - g.x;
        x[4 * S].x = u.x - g.y; x[4 * S].y = u.y + g.x;
        x[2 * S].x = v.x + h.y; x[2 * S].y = v.y - h.x;
        x[3 * S].x = v.x - h.y; x[3 * S].y = v.y + h.x;
    }
};

// Composite radix R = A B: with n = B n1 + n2 and k = k1 + A k2, DFTs of
// length A over n1, rotations by n2 k1 / R, DFTs of length B over n2; the
// last step moves the results to their order.
template <int A, int B, int N2, int K1, typename C>
__device__ __forceinline__ void comp_rot(C *x)
{
    if constexpr (N2 < B) {
        rot<N2 * K1, A * B>(x[B * K1 + N2]);
        if constexpr (K1 + 1 < A) comp_rot<A, B, N2, K1 + 1>(x);
        else comp_rot<A, B, N2 + 1, 1>(x);
    }
}
template <int A, int B, typename C> struct DftComp {
    template <int S> static __device__ __forceinline__ void go(C *x)
    {
        static_assert(S == 1, "composite radices work on adjacent values");
#pragma unroll
        for (int n2 = 0; n2 < B; ++n2) Dft<A, C>::template go<B>(x + n2);
        comp_rot<A, B, 1, 1>(x);  // x[B k1 + n2] holds (k1, n2)
#pragma unroll
        for (int k1 = 0; k1 < A; ++k1) Dft<B, C>::template go<1>(x + B * k1);
        C y[A * B];               // x[B k1 + k2] is output k1 + A k2
#pragma unroll
        for (int i = 0; i < A * B; ++i) y[i] = x[i];
#pragma unroll
        for (int k1 = 0; k1 < A; ++k1)
#pragma unroll
            for (int k2 = 0; k2 < B; ++k2) x[k1 + A * k2] = y[B * k1 + k2];
    }
};
template <typename C> struct Dft<6, C> : DftComp<2, 3, C> {};
template <typename C> struct Dft<8, C> : DftComp<2, 4, C> {};
template <typename C> struct Dft<9, C> : DftComp<3, 3, C> {};
template <typename C> struct Dft<10, C> : DftComp<2, 5, C> {};
template <typename C> struct Dft<12, C> : DftComp<3, 4, C> {};
template <typename C> struct Dft<15, C> : DftComp<3, 5, C> {};
template <typename C> struct Dft<16, C> : DftComp<4, 4, C> {};

// Skewed LDS position of element e of a line (stages store with strides that
// are multiples of 16).
__device__ __forceinline__ int skew(int e) { return e + (e >> 4); }

// Index of frequency l (mod n) among the N kept modes, negative when dropped.
__device__ __forceinline__ int mode_of(int l, int N, int n)
{
    // (a dropped l lies between the kept ends, where l - n + N / 2 < 0)
    return l <= N - 1 - N / 2 ? l + N / 2 : l - n + N / 2;
}

// Radices up to this one (a butterfly takes one thread's values).
constexpr int max_radix(int V) { return V < 16 ? V : 16; }

// The lines a block works on and where this thread stands in them.
struct Where {
    int t, c;          // thread of the line, line of the block
    bool on;           // the line exists
    int a;             // its first index
    long long src, dst;
};

// Forms of a pass: every element, the N kept modes of the outputs only
// (type 1), or of the inputs only (type 2).
enum { kWhole = 0, kCutOut = 1, kPadIn = 2 };

// What the stages need of a pass, loaded together when a block starts (the
// arguments are cold then; fetched where they are used, each stage waited for
// another line of them: 5.2-7.6 us a pass over a 128 x 128 grid after 6.4-8.4).
template <typename C>
struct Args {
    int n, np, T, pitch, inv, cut, scale, pe, pa, full;
    long long s_e, d_e;
    const void *fe;
    const C *tw, *tw4;
    unsigned long long radices;
    // The state of the stage loop: values per butterfly group so far, the
    // stage's first factor.
    int Ns, tw0;
};

template <typename T, int V, int FORM, typename C = typename Cplx<T>::type>
struct Stage {
    // One radix stage: B butterflies of R values per thread.
    template <int R>
    static __device__ __forceinline__ void go(const Args<C> &p, int q, Where &w, const Where &w2,
                                              T sab, const C *src, C *dst, C *lds)
    {
        constexpr int B = V / R;
        const bool first = q == 0, last = q == p.np - 1;
        const int nbf = p.n / R, Ns = p.Ns;
        // (j + 1/2) / Ns is at least 1 / (2 Ns) from an integer, j < 2^16
        const float rNs = 1.0f / (float)Ns;
        C x[B][R];
        int jm[B], jq[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int j = w.t + b * p.T;
            jq[b] = first ? j : (int)(((float)j + 0.5f) * rNs);  // j / Ns
            jm[b] = j - jq[b] * Ns;
            if (j >= nbf || !w.on) continue;
            if (first) {
                // element j + k nbf; frequencies l (mod full) in order, the
                // kept ones at i = l + N / 2 or, from the top, less by full
                if constexpr (FORM == kPadIn) {
                    // (loads first, all of them: dropped elements read the
                    // line's first mode and are cleared below)
                    const int N = p.cut, dl = nbf * p.pe, l0 = j * p.pe + w.a * p.pa;
                    const C *at = src + w.src;
                    T f[R];
#pragma unroll
                    for (int k = 0; k < R; ++k) {
                        const int i = mode_of(l0 + k * dl, N, p.full);
                        x[b][k] = at[(long long)max(i, 0) * p.s_e];
                    }
#pragma unroll
                    for (int k = 0; k < R; ++k) {
                        const int i = mode_of(l0 + k * dl, N, p.full);
                        f[k] = p.scale ? static_cast<const T *>(p.fe)[max(i, 0)] * sab : (T)1;
                        f[k] = i >= 0 ? f[k] : (T)0;
                        if (i < 0) x[b][k].x = x[b][k].y = (T)0;
                    }
#pragma unroll
                    for (int k = 0; k < R; ++k) {
                        const T re = x[b][k].x * f[k], im = x[b][k].y * f[k];
                        x[b][k].x = p.inv ? im : re;
                        x[b][k].y = p.inv ? re : im;
                    }
                } else {
                    const C *at = src + w.src + (long long)j * p.s_e;
                    const long long da = (long long)nbf * p.s_e;
#pragma unroll
                    for (int k = 0; k < R; ++k) {
                        const C v = *at;
                        x[b][k].x = p.inv ? v.y : v.x;
                        x[b][k].y = p.inv ? v.x : v.y;
                        at += da;
                    }
                }
            } else {
                // exp(-2 pi i jm k / (Ns R)), k = 1 .. R - 1, rows of Ns
                const C *f = p.tw + p.tw0 + jm[b];
#pragma unroll
                for (int k = 0; k < R; ++k) x[b][k] = lds[w.c * p.pitch + skew(j + k * nbf)];
#pragma unroll
                for (int k = 1; k < R; ++k) {
                    const C g = f[(k - 1) * Ns];
                    const T xr = x[b][k].x * g.x - x[b][k].y * g.y;
                    x[b][k].y = x[b][k].x * g.y + x[b][k].y * g.x;
                    x[b][k].x = xr;
                }
            }
            Dft<R, C>::template go<1>(x[b]);
        }
        if (!last) {
            if (!first) __syncthreads();  // every value of this stage has been read
#pragma unroll
            for (int b = 0; b < B; ++b) {
                if (w.t + b * p.T >= nbf || !w.on) continue;
                const int base = jq[b] * Ns * R + jm[b];
#pragma unroll
                for (int k = 0; k < R; ++k) lds[w.c * p.pitch + skew(base + k * Ns)] = x[b][k];
            }
            __syncthreads();
            if (first) w = w2;
            return;
        }
#pragma unroll
        for (int b = 0; b < B; ++b) {
            if (w.t + b * p.T >= nbf || !w.on) continue;
            const int base = jq[b] * Ns * R + jm[b];
            if constexpr (FORM != kCutOut) {
                if (p.tw4) {
                    // between the two halves of a long line: exp(-2 pi i a e / full)
                    int m = w.a * base;
#pragma unroll
                    for (int k = 0; k < R; ++k) {
                        const C f = p.tw4[m & (kTw4 - 1)];
                        const C g = p.tw4[kTw4 + m / kTw4];
                        const T fx = f.x * g.x - f.y * g.y, fy = f.x * g.y + f.y * g.x;
                        const T xr = x[b][k].x * fx - x[b][k].y * fy;
                        x[b][k].y = x[b][k].x * fy + x[b][k].y * fx;
                        x[b][k].x = xr;
                        m += w.a * Ns;
                    }
                }
            }
            if constexpr (FORM == kCutOut) {
                const int N = p.cut, dl = Ns * p.pe, l0 = base * p.pe + w.a * p.pa;
                C *at = dst + w.dst;
                T f[R];
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    const int i = mode_of(l0 + k * dl, N, p.full);
                    f[k] = p.scale ? sab * static_cast<const T *>(p.fe)[max(i, 0)] : (T)1;
                }
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    const int i = mode_of(l0 + k * dl, N, p.full);
                    C v;
                    v.x = (p.inv ? x[b][k].y : x[b][k].x) * f[k];
                    v.y = (p.inv ? x[b][k].x : x[b][k].y) * f[k];
                    if (i >= 0) at[(long long)i * p.d_e] = v;
                }
            } else {
                C *at = dst + w.dst + (long long)base * p.d_e;
                const long long da = (long long)Ns * p.d_e;
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    C v;
                    v.x = p.inv ? x[b][k].y : x[b][k].x;
                    v.y = p.inv ? x[b][k].x : x[b][k].y;
                    *at = v;
                    at += da;
                }
            }
        }
    }
};

// Lines of one pass; with TAB, block -> entry of a table (a batch), else p0.
template <typename T, int V, int FORM, bool TAB>
__global__ void __launch_bounds__(kFftThreads)
k_fft_lines(FftPass p0, const FftPass *__restrict__ tab, int ntab,
            const typename Cplx<T>::type *src, typename Cplx<T>::type *dst)
{
    using C = typename Cplx<T>::type;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    C *lds = reinterpret_cast<C *>(smem_raw);
    unsigned tile = (unsigned)xcd_block(blockIdx.x, gridDim.x);
    int ent = 0;
    if constexpr (TAB) {
        int lo = 0, hi = ntab - 1;
        while (lo < hi) {
            const int mid = lo + ((hi - lo + 1) >> 1);
            if (tab[mid].tile0 <= (int)tile) lo = mid; else hi = mid - 1;
        }
        ent = lo;
    }
    const FftPass &p = TAB ? tab[ent] : p0;
    if constexpr (TAB) tile -= (unsigned)p.tile0;
    const unsigned r = tile / (unsigned)p.ta, tr = r / (unsigned)p.nb;
    const int ta = (int)(tile - r * (unsigned)p.ta);
    const int b_idx = (int)(r - tr * (unsigned)p.nb);
    const auto place = [&](int col) {
        Where w;
        const unsigned tid = threadIdx.x;
        if (col) {  // (a power of two lines)
            w.c = (int)(tid & (unsigned)(p.C - 1));
            w.t = (int)(tid >> p.logC);
        } else {
            w.c = (int)(tid / (unsigned)p.T);
            w.t = (int)(tid - (unsigned)w.c * (unsigned)p.T);
        }
        w.a = ta * p.C + w.c;
        w.on = w.c < p.C && w.t < p.T && w.a < p.na;
        w.src = p.s0 + w.a * p.s_a + b_idx * p.s_b + tr * p.s_t;
        w.dst = p.d0 + w.a * p.d_a + b_idx * p.d_b + tr * p.d_t;
        return w;
    };
    Where w = place(p.col0);
    const Where w2 = place(p.col1);
    // factors of the other dimensions, the first dimension's first as the
    // correction kernels multiply (a pass that scales keeps its thread order)
    T sab = (T)1;
    if (p.scale && w.on) {
        if (p.fa) sab = static_cast<const T *>(p.fa)[w.a];
        if (p.fb) sab *= static_cast<const T *>(p.fb)[b_idx];
    }
    Args<C> g{p.n, p.np, p.T, p.pitch, p.inv, p.cut, p.scale, p.pe, p.pa, p.full, p.s_e, p.d_e,
              p.fe, static_cast<const C *>(p.tw), static_cast<const C *>(p.tw4), p.radices, 1, 0};
    // (keeps the loads here)
    asm volatile("" ::"s"(g.n), "s"(g.np), "s"(g.T), "s"(g.pitch), "s"(g.inv), "s"(g.cut),
                 "s"(g.scale), "s"(g.pe), "s"(g.pa), "s"(g.full), "s"(g.s_e), "s"(g.d_e),
                 "s"(g.fe), "s"(g.tw), "s"(g.tw4), "s"(g.radices));
    // The first stage's factors are ones and the last stage's come from memory
    // too: their lines are fetched beside the first loads, a line per thread,
    // so that the later stages find them in the cache.
    C warm = {0, 0};
    T warmf = (T)0;
    if (p.tw_len > 0) warm = g.tw[min((int)threadIdx.x * (128 / (int)sizeof(C)), p.tw_len - 1)];
    if (FORM == kCutOut && g.scale)
        warmf = static_cast<const T *>(
            g.fe)[min((int)threadIdx.x * (128 / (int)sizeof(T)), g.cut - 1)];
    for (int q = 0; q < g.np; ++q) {
        if (q == 1) asm volatile("" ::"v"(warm.x), "v"(warmf));
        const int R = (int)(g.radices >> (8 * q)) & 255;
        switch (R) {
#define MN_R(RR)                                                                           \
    case RR:                                                                               \
        if constexpr (RR <= max_radix(V))                                                  \
            Stage<T, V, FORM>::template go<RR>(g, q, w, w2, sab, src, dst, lds);           \
        break;
            MN_R(2) MN_R(3) MN_R(4) MN_R(5) MN_R(6) MN_R(8) MN_R(9) MN_R(10) MN_R(12) MN_R(15)
            MN_R(16)
#undef MN_R
        }
        if (q) g.tw0 += (R - 1) * g.Ns;
        g.Ns *= R;
    }
}

}  // namespace fft
}  // namespace mn
