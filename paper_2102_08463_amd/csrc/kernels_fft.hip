// Passes of the fine-grid FFT: radix stages, block shapes, twiddle tables and
// the dispatch to the line kernels (fft_kernels.h).
#include "internal.h"

#include <algorithm>

namespace mn {
namespace fft {
template <typename T, int V, bool TAB>
hipError_t launch(int form, const FftPass &p, const FftPass *tab, int ntab, long long tiles, int threads,
                  int lds, const void *src, void *dst, hipStream_t s);
#define MN_EXTERN(TT, VV, BB)                                                                 \
    extern template hipError_t launch<TT, VV, BB>(int, const FftPass &, const FftPass *, int,      \
                                                  long long, int, int, const void *, void *,  \
                                                  hipStream_t);
MN_EXTERN(float, 16, false) MN_EXTERN(float, 16, true) MN_EXTERN(float, 24, false)
MN_EXTERN(float, 8, false) MN_EXTERN(float, 4, false)
MN_EXTERN(double, 8, false) MN_EXTERN(double, 8, true)
#undef MN_EXTERN
}  // namespace fft

namespace {

template <typename T> struct Cplx;
template <> struct Cplx<float> { using type = float2; };
template <> struct Cplx<double> { using type = double2; };

constexpr int kRadices[] = {16, 15, 12, 10, 9, 8, 6, 5, 4, 3, 2};

// out[m] = exp(-2 pi i m step / n), m < cnt, evaluated in double.
template <typename T>
__global__ void k_twiddle(int cnt, long long step, double n, typename Cplx<T>::type *__restrict__ out)
{
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= cnt) return;
    double sn, cs;
    sincospi(2.0 * ((double)m * (double)step) / n, &sn, &cs);
    typename Cplx<T>::type v;
    v.x = (T)cs;
    v.y = (T)-sn;
    out[m] = v;
}

// The factors of every stage after the first: stage q holds, for k = 1 ..
// R - 1, a row of Ns values exp(-2 pi i j k / (Ns R)).
template <typename T>
__global__ void k_stage_twiddle(FftPass p, typename Cplx<T>::type *__restrict__ out)
{
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    for (int q = 0, Ns = 1, at = 0; q < p.np; ++q) {
        const int R = (int)(p.radices >> (8 * q)) & 255, e = m - at, len = q ? (R - 1) * Ns : 0;
        if (e >= 0 && e < len) {
            const int k = e / Ns + 1, j = e % Ns;
            double sn, cs;
            sincospi(2.0 * ((double)j * k) / ((double)Ns * R), &sn, &cs);
            typename Cplx<T>::type v;
            v.x = (T)cs;
            v.y = (T)-sn;
            out[m] = v;
        }
        at += len;
        Ns *= R;
    }
}

// Threads per line for radices R[0..np).
int threads_of(int n, const int *R, int np, int V)
{
    int T = 1;
    for (int q = 0; q < np; ++q) {
        const int per = V / R[q];
        T = std::max(T, (n / R[q] + per - 1) / per);
    }
    return T;
}

// Radices of n: fewest stages, then fewest threads per line.
void search(int n, int rest, int maxr, int np, int *R, int V, int *best, int &bnp, int &bT)
{
    if (rest == 1) {
        const int T = threads_of(n, R, np, V);
        if (bnp == 0 || np < bnp || (np == bnp && T < bT)) {
            bnp = np;
            bT = T;
            std::copy(R, R + np, best);
        }
        return;
    }
    if (np == kFftStages || (bnp && np + 1 > bnp)) return;
    for (int r : kRadices) {
        if (r > maxr || rest % r) continue;
        R[np] = r;
        search(n, rest / r, r, np + 1, R, V, best, bnp, bT);
    }
}

}  // namespace

bool fft_line(int n, int V, FftPass &p)
{
    int R[kFftStages] = {}, best[kFftStages] = {}, np = 0, T = 0;
    if (n < 2) return false;
    search(n, n, std::min(V, 16), 0, R, V, best, np, T);
    if (np == 0) return false;
    p.n = n;
    p.np = np;
    p.T = T;
    p.radices = 0;
    p.tw_len = 0;
    for (int q = 0, Ns = 1; q < np; ++q) {
        p.radices |= (unsigned long long)best[q] << (8 * q);
        if (q) p.tw_len += (best[q] - 1) * Ns;
        Ns *= best[q];
    }
    return true;
}

// Lines per block.  Row passes (the line is contiguous) aim at 256 threads;
// column passes at 64 B or more per row of a tile (128 B where two blocks
// still fit a CU), as adjacent tiles share the rest of a cache line in L2.
// Both take fewer lines per block while the pass has under 512 blocks, down
// to one wave (rows) or 32 B (columns).  False when no choice keeps 32 B.
bool fft_tile(FftPass &p, int prec, bool rows, long long outer)
{
    const size_t csz = prec == 0 ? 8 : 16;
    const int unit = (int)(32 / csz);  // lines of a 32 B piece
    const auto bytes = [&](int C) {
        int pitch = p.n + p.n / 16 + 1;
        if (C <= 16) {
            const int want = 16 / C % 16;
            pitch += ((want - pitch) % 16 + 16) % 16;
        }
        p.pitch = pitch;
        return (size_t)pitch * C * csz;
    };
    int na2 = 1;
    while (na2 < p.na) na2 *= 2;
    int C = 1;
    if (rows) {
        while (2 * C * p.T <= 256 && C < na2) C *= 2;
    } else {
        C = std::min(4 * unit, na2);
        while (C > 2 * unit && bytes(C) > 80 * 1024) C /= 2;
    }
    while (C > 1 && (C * p.T > kFftThreads || bytes(C) > 160 * 1024)) C /= 2;
    const int least = rows ? std::max(1, 64 / p.T) : std::min(unit, na2);
    while (C / 2 >= least && (long long)((p.na + C - 1) / C) * outer < 512) C /= 2;
    if (C * p.T > kFftThreads || bytes(C) > 160 * 1024) return false;
    if (!rows && C < std::min(unit, na2)) return false;
    p.C = C;
    p.logC = 0;
    while ((1 << p.logC) < C) ++p.logC;
    p.lds = (int)bytes(C);
    p.ta = (p.na + C - 1) / C;
    p.threads = (C * p.T + 63) / 64 * 64;
    return true;
}

hipError_t launch_twiddle(int prec, int cnt, long long step, double n, void *out, hipStream_t s)
{
    if (cnt <= 0) return hipSuccess;
    const dim3 g((cnt + 255) / 256), b(256);
    if (prec == 0)
        hipLaunchKernelGGL(k_twiddle<float>, g, b, 0, s, cnt, step, n, (float2 *)out);
    else
        hipLaunchKernelGGL(k_twiddle<double>, g, b, 0, s, cnt, step, n, (double2 *)out);
    return hipGetLastError();
}

hipError_t launch_stage_twiddle(int prec, const FftPass &p, void *out, hipStream_t s)
{
    if (p.tw_len <= 0) return hipSuccess;
    const dim3 g((p.tw_len + 255) / 256), b(256);
    if (prec == 0)
        hipLaunchKernelGGL(k_stage_twiddle<float>, g, b, 0, s, p, (float2 *)out);
    else
        hipLaunchKernelGGL(k_stage_twiddle<double>, g, b, 0, s, p, (double2 *)out);
    return hipGetLastError();
}

hipError_t launch_fft_lines(int prec, int V, int form, const FftPass &p, const FftPass *tab, int ntab,
                            long long tiles, int threads, int lds, const void *src, void *dst,
                            hipStream_t s)
{
    if (tiles <= 0) return hipSuccess;
    if (tiles > 2147483647LL || threads > kFftThreads ||
        (tab && V != fft_values(prec))) return hipErrorInvalidValue;
#define MN_GO(TT, VV, BB) fft::launch<TT, VV, BB>(form, p, tab, ntab, tiles, threads, lds, src, dst, s)
    if (prec == 0) {
        if (V == 24) return MN_GO(float, 24, false);
        if (V == 4) return MN_GO(float, 4, false);
        if (V == 8) return MN_GO(float, 8, false);
        return tab ? MN_GO(float, 16, true) : MN_GO(float, 16, false);
    }
    return tab ? MN_GO(double, 8, true) : MN_GO(double, 8, false);
#undef MN_GO
}

}  // namespace mn
