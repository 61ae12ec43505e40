// Matrix-core spreading and interpolation of method SM, double precision 3D.
//
// A tap-by-tap kernel touches w^d cells per point: at w = 13 that is 2 x 2197
// 64-bit LDS atomics (spreading) or 2197 16-byte LDS reads (interpolation) per
// point, and both were bound by them.  Here the points of a subproblem are
// kept in groups (k_group): a group's points start, per dimension, within
// s = 17 - w cells of each other, so all their taps lie in one window of 16
// cells per dimension, and a window is a dense contraction over its points:
//   spreading      win[z][y][x] = sum_j (kz_j[z] ky_j[y]) (kx_j[x] c_j)
//   interpolation  v_j = sum_x kx_j[x] sum_{z,y} (kz_j[z] ky_j[y]) win[z][y][x]
// with the kernel values placed at the point's taps and exact zeros elsewhere.
// v_mfma_f64_16x16x4 does 1024 FMAs in 64 cycles of a SIMD; the window has
// 16^3 / w^3 times the cells (1.9 at w = 13), and a window's sums go to the
// tile once per group, not once per point.  An infinity or NaN times such a zero
// would reach the whole window: strengths and tiles that hold one take the
// points tap by tap.
#pragma once
#include "spread_kernels.h"

namespace mn {
namespace detail {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kMfThreads = 512;   // spreading: two waves per SIMD; the tile fills a CU's LDS
constexpr int kMfPts = 32;        // points whose kernel values are staged at a time
constexpr int kMfInterp = 1024;   // interpolation: four waves per SIMD
constexpr int kMfPart = 1024;     // points of a work item of interpolation
constexpr int kMfBlocks = 256;    // one per CU
constexpr int kMfOdd = 1 << 30;   // with a point's window origin: strength not finite

// Work items handed out one at a time: a block per CU fits, items differ by a
// factor of 4096 in size, and a fixed share left a fifth of the CUs idle at
// the end.  next() returns the block's next item, `total` or more when none is
// left, and leaves the counter at zero for the next launch: every block asks
// until it is refused, so the last refusal is number total + blocks - 1.
// (All threads call it; it holds a barrier, and the one before the returned
// item's shared memory is written.)
struct WorkQueue {
    int *counter;
    int *slot;   // shared memory
    __device__ __forceinline__ int next(int total) const
    {
        __syncthreads();
        if (threadIdx.x == 0) {
            const int i = atomicAdd(counter, 1);
            if (i == total + (int)gridDim.x - 1) atomicExch(counter, 0);
            *slot = i;
        }
        __syncthreads();
        return *slot;
    }
};

// Kernel value at slot `slot` of a window whose origin lies `off` cells before
// the point's first tap; z0 as in tap_start.
template <int W>
__device__ __forceinline__ double slot_val(double z0, int slot, int off, double bk)
{
    const int a = slot - off;
    const double v = es_val(z0 + (double)a * (2.0 / W), bk);
    return (a >= 0 && a < W) ? v : 0.0;
}

// Start of a point's taps in its padded tile and z0 of the first.
template <int W>
__device__ __forceinline__ int start_of(double u, double &z0)
{
    constexpr int P = (W + 1) / 2;
    return tap_start<double, W>(u + (double)P, z0);
}

// Spreading.  Wave v owns the tile planes whose z is 2 v or 2 v + 1 modulo 16,
// whatever the group, and computes those of each window: its sums go to the
// tile by plain adds that no other wave touches, in point order, so the tile
// is reproducible without fixed point.  The block evaluates 32 points' kernel
// values at a time (one slot of each dimension per thread, the strength
// multiplied into x) while the next points' loads are in flight.  Double
// precision vector instructions and matrix instructions share the pipe
// (evaluating in extra waves beside the products was slower: 11.5 ms for 9.9),
// so what is left beside the products is kept short: each step of four points
// reads five operands and multiplies two.  w = 13, 1.6e7 points in caps on
// 162^3: 33.0 -> 7.0 ms; the products alone would take 3.6 ms.
template <int W>
__global__ void __launch_bounds__(kMfThreads)
k_spread_mf(Geom g, const int32_t *__restrict__ sub, const int32_t *__restrict__ nsubp,
            const double *__restrict__ u0, const double *__restrict__ u1,
            const double *__restrict__ u2, const int32_t *__restrict__ idx,
            const double2 *__restrict__ c, double2 *__restrict__ scratch, int tcells, double bk,
            int *__restrict__ work, int nt, TStride tst)
{
    __shared__ int next_item;
    const WorkQueue queue{work, &next_item};
    constexpr int P = (W + 1) / 2, S = 17 - W;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    double2 *tile = reinterpret_cast<double2 *>(smem_raw);
    // per staged point 16 slots each of Re(c) kx, Im(c) kx, ky, kz; origins
    double *wts = reinterpret_cast<double *>(tile + tcells);
    int *org = reinterpret_cast<int *>(wts + kMfPts * 64);
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int sl = lane & 15, kp = lane >> 4;
    const int p1 = g.m[0] + 2 * P, p2 = g.m[1] + 2 * P, p3 = g.m[2] + 2 * P;
    const int nsub = *nsubp;
    for (int it = queue.next(nsub * nt); it < nsub * nt; it = queue.next(nsub * nt)) {
        const int tr = it / nsub, q = it - tr * nsub;  // stacked transform, subproblem
        const int4 rec = reinterpret_cast<const int4 *>(sub)[q];
        const double2 *ct = c + tr * tst.c;
        const int end = rec.y + rec.z;
        for (int e = tid; e < tcells; e += kMfThreads) tile[e] = make_double2(0.0, 0.0);
        // this thread's point of a chunk, clamped to the subproblem
        const auto at = [&](int i0) { return min(i0 + (tid >> 4), end - 1); };
        int ci = idx[at(rec.y)];
        double nu0 = u0[at(rec.y)], nu1 = u1[at(rec.y)], nu2 = u2[at(rec.y)];
        double2 nc = ct[ci];
        ci = idx[at(rec.y + kMfPts)];
        d4 ar0 = {0, 0, 0, 0}, ai0 = {0, 0, 0, 0}, ar1 = {0, 0, 0, 0}, ai1 = {0, 0, 0, 0};
        int cur = -1, z0a = 0, z0b = 0;
        const auto flush = [&]() {
            const int ox = cur & 255, oy = (cur >> 8) & 255, oz = cur >> 16;
            const int X = ox + sl;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int Z = oz + (h ? z0b : z0a);
                const d4 r = h ? ar1 : ar0, i = h ? ai1 : ai0;
                // all reads first (for cells past the tile: its last one)
                double2 v[4];
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    v[k] = tile[(min(Z, p3 - 1) * p2 + min(oy + 4 * k + kp, p2 - 1)) * p1 +
                                min(X, p1 - 1)];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int Y = oy + 4 * k + kp;
                    v[k].x += r[k];
                    v[k].y += i[k];
                    if (Z < p3 && Y < p2 && X < p1) tile[(Z * p2 + Y) * p1 + X] = v[k];
                }
            }
            ar0 = ai0 = ar1 = ai1 = d4{0, 0, 0, 0};
        };
        for (int i0 = rec.y; i0 < end; i0 += kMfPts) {
            {
                const int pt = tid >> 4, slot = tid & 15;
                double *w = wts + pt * 64 + slot;
                double z0;
                int st = start_of<W>(nu0, z0), og = st / S * S, o = og;
                const double kx = slot_val<W>(z0, slot, st - og, bk);
                w[0] = kx * nc.x;
                w[16] = kx * nc.y;
                st = start_of<W>(nu1, z0), og = st / S * S, o |= og << 8;
                w[32] = slot_val<W>(z0, slot, st - og, bk);
                st = start_of<W>(nu2, z0), og = st / S * S, o |= og << 16;
                w[48] = slot_val<W>(z0, slot, st - og, bk);
                if (!isfinite(nc.x) || !isfinite(nc.y)) {
                    o |= kMfOdd;  // (in segments of their own, see below)
                    if (kx == 0.0) w[0] = w[16] = 0.0;
                }
                if (slot == 0) org[pt] = o;
            }
            nu0 = u0[at(i0 + kMfPts)];
            nu1 = u1[at(i0 + kMfPts)];
            nu2 = u2[at(i0 + kMfPts)];
            nc = ct[ci];
            ci = idx[at(i0 + 2 * kMfPts)];
            __syncthreads();
            const int nv = min(kMfPts, end - i0);
            const int mine = org[min(lane, nv - 1)];
            const int prev = __shfl_up(mine, 1, 64);
            const uint64_t edge = __ballot(lane > 0 && lane < nv && mine != prev);
            for (int a = 0; a < nv;) {
                const uint64_t rest = edge & (~0ull << (a + 1));
                const int b = rest ? (int)__builtin_ctzll(rest) : nv;
                const int og = __builtin_amdgcn_readlane(mine, a);
                if (og & kMfOdd) {
                    // cells of the point's support alone, in this wave's planes
                    const int ox = og & 255, oy = (og >> 8) & 255, oz = (og >> 16) & 255;
                    for (int e = a * 2; e < b * 2; ++e) {
                        const double *w = wts + (e >> 1) * 64;
                        const int z = (2 * wv + (e & 1) - oz) & 15, Z = oz + z, X = ox + sl;
                        for (int k = 0; k < 4; ++k) {
                            const int y = 4 * k + kp, Y = oy + y;
                            const double f = w[32 + y] * w[48 + z];
                            if (f != 0.0 && (w[sl] != 0.0 || w[16 + sl] != 0.0)) {
                                double2 &t = tile[(Z * p2 + Y) * p1 + X];
                                t.x += f * w[sl];
                                t.y += f * w[16 + sl];
                            }
                        }
                    }
                    a = b;
                    continue;
                }
                if (og != cur) {
                    if (cur >= 0) flush();
                    cur = og;
                    z0a = (2 * wv - (og >> 16)) & 15;
                    z0b = (2 * wv + 1 - (og >> 16)) & 15;
                }
                const auto step = [&](const double *w, const double *za, const double *zb,
                                      bool on) {
                    double br = w[0], bi = w[16];
                    const double ky = w[32], a0 = ky * za[0], a1 = ky * zb[0];
                    if (!on) br = bi = 0.0;
                    ar0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, br, ar0, 0, 0, 0);
                    ai0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, bi, ai0, 0, 0, 0);
                    ar1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, br, ar1, 0, 0, 0);
                    ai1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, bi, ai1, 0, 0, 0);
                };
                const double *w = wts + (a + kp) * 64 + sl;
                const double *za = wts + (a + kp) * 64 + 48 + z0a, *zb = za + (z0b - z0a);
                int i = a;
                for (; i + 4 <= b; i += 4, w += 256, za += 256, zb += 256) step(w, za, zb, true);
                if (i < b) {
                    // the last points of the segment (past them: no strength)
                    const bool on = i + kp < b;
                    const int back = on ? 0 : (i + kp - (b - 1)) * 64;
                    step(w - back, za - back, zb - back, on);
                }
                a = b;
            }
            __syncthreads();  // the staged values are no longer read
        }
        if (cur >= 0) flush();
        __syncthreads();
        double2 *dst = scratch + tr * (tst.tiles / 2) + (size_t)q * tcells;
        for (int e = tid; e < tcells; e += kMfThreads) dst[e] = tile[e];
    }
}

// Interpolation.  The padded bin is staged in LDS; each wave takes a
// contiguous share of the item's points, sixteen of one group at a time
// as the rows of the products.  A lane evaluates the kernel values it
// multiplies with: four slots of ky and kz of its row's point and of kx of
// the four points it reduces; the other z slots come by lane shuffles.
// w = 13, 1.0e6 points in caps on 90^3: 1.78 -> 0.75 ms, products alone 0.26.
template <int W>
__global__ void __launch_bounds__(kMfInterp)
k_interp_mf(Geom g, const int32_t *__restrict__ sub, const int32_t *__restrict__ nsubp,
            const double *__restrict__ u0, const double *__restrict__ u1,
            const double *__restrict__ u2, const int32_t *__restrict__ idx,
            const double2 *__restrict__ grid, double2 *__restrict__ c, double bk,
            int *__restrict__ work, int nt, TStride tst)
{
    __shared__ int next_item;
    const WorkQueue queue{work, &next_item};
    constexpr int P = (W + 1) / 2, S = 17 - W;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    double2 *tile = reinterpret_cast<double2 *>(smem_raw);
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int sl = lane & 15, kp = lane >> 4;
    const int p1 = g.m[0] + 2 * P, p2 = g.m[1] + 2 * P, p3 = g.m[2] + 2 * P;
    const int nsub = *nsubp;
    // work item = kMfPart points of a subproblem (at most 4096 points, so most
    // of the later parts are empty)
    const int items = 4096 / kMfPart * nsub * nt;
    __shared__ int odd[2];  // the staged tile holds values that are not finite; item by item
    int turn = 0;
    if (tid < 2) odd[tid] = 0;  // (the queue's barriers come before their use)
    // A counter serves one launch at a time; one that may run beside another of
    // its plan has none and takes every gridDim-th item.
    const auto next = [&](int it) {
        if (work) return queue.next(items);
        __syncthreads();
        return it < 0 ? (int)blockIdx.x : it + (int)gridDim.x;
    };
    for (int it = next(-1); it < items; it = next(it)) {
        const int pt = it / nsub, part = pt / nt, tr = pt - part * nt;
        const double2 *gt = grid + tr * tst.grid;
        double2 *ct = c + tr * tst.c;
        int4 rec = reinterpret_cast<const int4 *>(sub)[it - pt * nsub];
        rec.y += part * kMfPart;
        rec.z = min(rec.z - part * kMfPart, kMfPart);
        if (rec.z <= 0) continue;
        const int b1 = rec.x % g.B[0], b23 = rec.x / g.B[0];
        const int b2 = b23 % g.B[1], b3 = b23 / g.B[1];
        const int o1 = b1 * g.m[0] - P, o2 = b2 * g.m[1] - P, o3 = b3 * g.m[2] - P;
        // rows of the padded bin, 32 lanes each, eight rows' loads in flight
        constexpr int kRows = 8, kStep = kMfInterp / 32;
        const int rows = p2 * p3;
        for (int s1 = lane & 31; s1 < p1; s1 += 32) {
            const int l1 = wrapmod(o1 + s1, g.n[0]);
            for (int r0 = tid >> 5; r0 < rows; r0 += kRows * kStep) {
                double2 v[kRows];
#pragma unroll
                for (int k = 0; k < kRows; ++k) {
                    const int r = min(r0 + k * kStep, rows - 1), s3 = r / p2, s2 = r - s3 * p2;
                    v[k] = gt[((size_t)wrapmod(o3 + s3, g.n[2]) * g.n[1] +
                                 wrapmod(o2 + s2, g.n[1])) * g.n[0] + l1];
                }
#pragma unroll
                for (int k = 0; k < kRows; ++k) {
                    if (r0 + k * kStep < rows) tile[(r0 + k * kStep) * p1 + s1] = v[k];
                    if (!isfinite(v[k].x) || !isfinite(v[k].y)) odd[turn] = 1;
                }
            }
        }
        __syncthreads();
        const int tap_by_tap = odd[turn];
        turn ^= 1;
        if (tid == 0) odd[turn] = 0;
        if (tap_by_tap) {
            for (int i = rec.y + tid; i < rec.y + rec.z; i += kMfInterp) {
                double zy, zz, ar = 0.0, ai = 0.0, kx[W];
                const int sx = taps<double, W>(u0[i] + (double)P, bk, kx);
                const int sy = start_of<W>(u1[i], zy), sz = start_of<W>(u2[i], zz);
#pragma unroll 1
                for (int a3 = 0; a3 < W; ++a3) {
                    const double kz = es_val(zz + (double)a3 * (2.0 / W), bk);
#pragma unroll 1
                    for (int a2 = 0; a2 < W; ++a2) {
                        const double f = kz * es_val(zy + (double)a2 * (2.0 / W), bk);
                        const double2 *row = tile + ((sz + a3) * p2 + sy + a2) * p1 + sx;
                        double rr = 0.0, ri = 0.0;
#pragma unroll
                        for (int a1 = 0; a1 < W; ++a1) {
                            rr += kx[a1] * row[a1].x;
                            ri += kx[a1] * row[a1].y;
                        }
                        ar += f * rr;
                        ai += f * ri;
                    }
                }
                ct[idx[i]] = make_double2(ar, ai);
            }
            continue;
        }
        const int share = (rec.z + kMfInterp / 4 - 1) / (kMfInterp / 4) * 16;  // points per wave
        const int w0 = rec.y + wv * share, w1 = min(w0 + share, rec.y + rec.z);
        for (int i0 = w0; i0 < w1; i0 += 64) {
            const int nv = min(64, w1 - i0), il = i0 + min(lane, nv - 1);
            const double x0 = u0[il], x1 = u1[il], x2 = u2[il];
            const int pj = idx[il];
            double zx, zy, zz;
            const int sx = start_of<W>(x0, zx), sy = start_of<W>(x1, zy), sz = start_of<W>(x2, zz);
            const int mine = (sx / S * S) | ((sy / S * S) << 8) | ((sz / S * S) << 16);
            const int fx = sx % S, fy = sy % S, fz = sz % S;
            const int prev = __shfl_up(mine, 1, 64);
            const uint64_t edge = __ballot(lane > 0 && lane < nv && mine != prev);
            for (int a = 0; a < nv;) {
                const uint64_t rest = a + 1 < 64 ? edge & (~0ull << (a + 1)) : 0ull;
                const int b = min(rest ? (int)__builtin_ctzll(rest) : nv, a + 16);
                const int og = __builtin_amdgcn_readfirstlane(__shfl(mine, a, 64));
                const int ox = og & 255, oy = (og >> 8) & 255, oz = og >> 16;
                // kernel values: row point sl at slots 4 i + kp of y and z
                const int pr = min(a + sl, b - 1);
                const double ry = __shfl(zy, pr, 64), rz = __shfl(zz, pr, 64);
                const int gy = __shfl(fy, pr, 64), gz = __shfl(fz, pr, 64);
                double ky[4], kz[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    ky[i] = slot_val<W>(ry, 4 * i + kp, gy, bk);
                    kz[i] = slot_val<W>(rz, 4 * i + kp, gz, bk);
                }
                d4 tr = {0, 0, 0, 0}, ti = {0, 0, 0, 0};
                const int X = min(ox + sl, p1 - 1);
                const int nz = min(16, p3 - oz);
#pragma unroll
                for (int zq = 0; zq < 4; ++zq) {
                    for (int zl = 0; zl < 4; ++zl) {
                        const int z = 4 * zq + zl;
                        if (z >= nz) break;
                        const double kzv = __shfl(kz[zq], zl * 16 + sl, 64);
                        const double2 *pl = tile + (size_t)(oz + z) * p2 * p1 + X;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const double2 v = pl[min(oy + 4 * i + kp, p2 - 1) * p1];
                            const double f = ky[i] * kzv;
                            tr = __builtin_amdgcn_mfma_f64_16x16x4f64(f, v.x, tr, 0, 0, 0);
                            ti = __builtin_amdgcn_mfma_f64_16x16x4f64(f, v.y, ti, 0, 0, 0);
                        }
                    }
                }
                // lane holds rows 4 k + kp at column sl: times kx, summed over columns
                double2 res = make_double2(0.0, 0.0);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int po = min(a + 4 * k + kp, b - 1);
                    const double kx = slot_val<W>(__shfl(zx, po, 64), sl, __shfl(fx, po, 64), bk);
                    double vr = tr[k] * kx, vi = ti[k] * kx;
#pragma unroll
                    for (int o = 8; o > 0; o >>= 1) {
                        vr += __shfl_xor(vr, o, 64);
                        vi += __shfl_xor(vi, o, 64);
                    }
                    if (sl == k) res = make_double2(vr, vi);
                }
                const int row = a + 4 * sl + kp;  // (sl < 4) the point of res
                const int dst = __shfl(pj, min(row, 63), 64);
                if (sl < 4 && row < b) ct[dst] = res;
                a = b;
            }
        }
    }
}

template <int W>
hipError_t spread_mf(const Geom &g, const Pts &P, const void *c, hipStream_t s)
{
    auto k = k_spread_mf<W>;
    const size_t lds = mf_lds_bytes(g) - 64;  // (what is not static)
    (void)hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(k, dim3(kMfBlocks), dim3(kMfThreads), lds, s, g, P.sub, P.nsub,
                       (const double *)P.u[0], (const double *)P.u[1], (const double *)P.u[2],
                       sm_index(P), (const double2 *)c, (double2 *)P.scratch, P.ts2 / 2,
                       kernel_param<double>(g.beta), P.work, P.nt,
                       TStride{(size_t)P.M, (size_t)P.ncells, P.tile_stride});
    return hipGetLastError();
}

template <int W>
hipError_t interp_mf(const Geom &g, const Pts &P, const void *grid, void *c, hipStream_t s)
{
    auto k = k_interp_mf<W>;
    const size_t lds = (size_t)sm_tile_stride(g) * 8;
    (void)hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(k, dim3(kMfBlocks), dim3(kMfInterp), lds, s, g, P.sub, P.nsub,
                       (const double *)P.u[0], (const double *)P.u[1], (const double *)P.u[2],
                       sm_index(P), (const double2 *)grid, (double2 *)c,
                       kernel_param<double>(g.beta), P.work ? P.work + 1 : nullptr, P.nt,
                       TStride{(size_t)P.M, (size_t)P.ncells, 0});
    return hipGetLastError();
}

}  // namespace detail
}  // namespace mn
