// Bin-sort of the nonuniform points (Sec. III-A, GM-sort and SM step 1).
//
// A point lies in the bin that holds its integer fine-grid coordinates
// l_i = floor((x_i + pi) / h_i).  The permutation t lists bin 0's points
// first, then bin 1's, ...; inside a bin the input order is kept, which makes
// t unique and reproducible.  It is built as a stable LSD radix sort of
// (bin key, input index) pairs with 8-bit digits: per pass a digit histogram
// per 4096-key tile, one exclusive scan over the (digit, tile) counts, and a
// scatter whose in-tile ranks come from wavefront ballots (all lanes holding
// the same digit are found with eight 64-bit ballots, so no lane order has to
// be assumed of LDS atomics).
//
// The grid coordinate is evaluated with a fixed sequence of correctly rounded
// double operations and no contraction: g = (x + pi) * S with S = n / (2 pi)
// rounded once on the host; then one whole-period correction.  That makes
// the keys, and hence t, reproducible bit for bit on any IEEE machine.
#include "internal.h"

#include <algorithm>
#include <type_traits>

namespace mn {
namespace {

constexpr double kPi = 3.141592653589793;
constexpr int kThreads = 256;
constexpr int kItems = 16;
constexpr int kTile = kThreads * kItems;  // keys per radix block
constexpr int kTileSmall = 1024;          // the same for at most kSmallKeys keys, which
constexpr int kSmallKeys = 1 << 20;       // would fill too few large blocks
// Up to this many blocks each scatter block sums the digit counts it needs
// itself (M = 1e5: the two scan launches took 9 us of a 55 us sort).
constexpr int kFusedBlocks = 256;
// Passes that move three single-precision planes of a sorted order take twice
// the tile: its longer digit runs write fewer partial lines (1.7e7 points, 128
// digits: 243 -> 203 us; the passes from the points and those of one or two
// planes got 10 to 20% slower with it).
constexpr int kTileWide = 2 * kTile;
inline int tile_of(int M, bool wide = false)
{
    return M <= kSmallKeys ? kTileSmall : (wide ? kTileWide : kTile);
}
// Distance between the digits' rows of counts.
inline int hist_pitch(int nblk) { return nblk <= kFusedBlocks ? (nblk + 3) / 4 * 4 : nblk; }

// Folded grid coordinate in [0, n).  `bad` is set when one period shift does
// not bring the value into range (non-finite or beyond about [-3pi, 3pi)).
__device__ __forceinline__ double grid_coord(double x, double S, int n, int &bad)
{
    const double nd = (double)n;
    double g = __dmul_rn(__dadd_rn(x, kPi), S);
    if (g < 0.0) g = __dadd_rn(g, nd);
    if (g >= nd) g = __dsub_rn(g, nd);
    if (!(g >= 0.0 && g < nd)) {
        bad = 1;
        const double q = floor(__ddiv_rn(g, nd));
        g = __dsub_rn(g, __dmul_rn(q, nd));
        if (g >= nd) g = __dsub_rn(g, nd);
        if (!(g >= 0.0 && g < nd)) g = 0.0;
    }
    return g;
}

// Bin key of point j and its bin-relative coordinates u[0..dim-1]; bad is
// set when a coordinate needed a fallback fold.  For a batch (BATCH), the
// point's transform is found among the pt_off values (soff: an LDS copy when
// cached, else the table itself).
// (xv: the point's coordinates, already loaded; unused dimensions ignored)
template <typename T, bool BATCH>
__device__ __forceinline__ uint32_t point_key_of(const Geom &g, const T xc[3], const PtMap &map,
                                                 const TGeom *tg, int T_, const long long *soff,
                                                 bool cached, int j, T u[3], int &bad)
{
    uint32_t k = 0, stride = 1;
    Geom gg = g;
    [[maybe_unused]] int own[2] = {0, 0};
    [[maybe_unused]] double own_im[2] = {0, 0};
    if constexpr (BATCH) {
        const auto fld = [](const TGeom &a) { return a.pt_off; };
        const int t = cached ? find_cached(soff, T_, j) : find_transform(tg, T_, j, fld);
        gg = geom_of(g, tg[t]);
        k = (uint32_t)tg[t].bin_off;
        if constexpr (std::is_same<T, float>::value)
            for (int d = 0; d < 2; ++d) {
                own[d] = tg[t].own[d];
                own_im[d] = tg[t].own_im[d];
            }
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        u[d] = (T)0;
        if (d >= gg.dim) continue;
        double xv = (double)xc[d];
        if (map.on) xv = __dmul_rn(__dsub_rn(xv, map.off[d]), map.mul[d]);
        const double gc = grid_coord(xv, gg.S[d], gg.n[d], bad);
        const int l = (int)gc;  // gc >= 0, so truncation is floor; l <= n - 1
        // l / m, exactly: (l + 1/2) / m is at least 1 / (2 m) from an integer
        const int b = (int)(((double)l + 0.5) * gg.im[d]);
        k += (uint32_t)b * stride;
        stride *= (uint32_t)gg.B[d];
        u[d] = (T)(gc - (double)b * (double)gg.m[d]);
        if constexpr (BATCH && std::is_same<T, float>::value) {
            if (d < 2 && own[d] > 0) {
                const int c = (int)(((double)l + 0.5) * own_im[d]) * own[d];  // own bin's first cell
                u[d] = __int_as_float(
                    fix_coord((float)(gc - (double)c), gg.pad, c - b * gg.m[d]));
            }
        }
    }
    return k;
}

template <typename T, bool BATCH>
__device__ __forceinline__ uint32_t point_key(const Geom &g, const T *x, const T *y, const T *z,
                                              const PtMap &map, const TGeom *tg, int T_,
                                              const long long *soff, bool cached, int j, T u[3],
                                              int &bad)
{
    const T xc[3] = {x[j], g.dim >= 2 ? y[j] : (T)0, g.dim == 3 ? z[j] : (T)0};
    return point_key_of<T, BATCH>(g, xc, map, tg, T_, soff, cached, j, u, bad);
}

template <typename T, bool BATCH>
__global__ void __launch_bounds__(kThreads)
k_binkey(Geom g, int M, const T *__restrict__ x, const T *__restrict__ y,
         const T *__restrict__ z, uint32_t *__restrict__ key, T *__restrict__ u0,
         T *__restrict__ u1, T *__restrict__ u2, int *__restrict__ flag,
         const TGeom *__restrict__ tg, int T_, PtMap map)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    __shared__ long long soff[BATCH ? kTCache : 1];
    bool cached = false;
    if constexpr (BATCH) cached = cache_offsets(soff, tg, T_, [](const TGeom &a) { return a.pt_off; });
    if (j >= M) return;
    int bad = 0;
    T u[3];
    const uint32_t k = point_key<T, BATCH>(g, x, y, z, map, tg, T_, soff, cached, j, u, bad);
    T *us[3] = {u0, u1, u2};
#pragma unroll
    for (int d = 0; d < 3; ++d)
        if (d < g.dim) us[d][j] = u[d];
    key[j] = k;
    if (bad) atomicOr(flag, 1);
}

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v, int lane)
{
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(v, o, 64);
        if (lane >= o) v += t;
    }
    return v;
}

// The transforms that points [j0, j1] of a batch belong to, as a table and
// its length: the points of a tile then search a few entries, not all.
__device__ __forceinline__ const TGeom *tile_transforms(const TGeom *tg, int &T_, int64_t j0,
                                                        int64_t j1)
{
    const auto fld = [](const TGeom &a) { return a.pt_off; };
    const int a = find_transform(tg, T_, j0, fld), b = find_transform(tg, T_, j1, fld);
    T_ = b - a + 1;
    return tg + a;
}

// A block's digit counts to column blockIdx.x; the last block also clears the
// columns up to the row pitch.
__device__ __forceinline__ void store_counts(const uint32_t *h, int pitch, uint32_t *hist)
{
    if (threadIdx.x >= 256) return;
    uint32_t *row = hist + (int64_t)threadIdx.x * pitch;
    row[blockIdx.x] = h[threadIdx.x];
    if (blockIdx.x == gridDim.x - 1)
        for (int k = gridDim.x; k < pitch; ++k) row[k] = 0u;
}

// Digit histogram of the first radix pass straight from the points (keys
// computed as point_key does; the validation flag set as k_binkey sets it).
// (1024 threads, kTile / 1024 points each: the key arithmetic is long, so
// more points are in flight per tile than with k_radix_hist's layout)
constexpr int kSrcThreads = 1024;
template <typename T, bool BATCH, int TILE>
__global__ void __launch_bounds__(kSrcThreads)
k_radix_hist_src(KeySrc src, int M, int shift, uint32_t dmask, int pitch,
                 uint32_t *__restrict__ hist)
{
    constexpr int kSrcItems = TILE / kSrcThreads;
    __shared__ uint32_t h[256];
    const int tid = threadIdx.x;
    if (tid < 256) h[tid] = 0;
    if constexpr (BATCH)
        src.tg = tile_transforms(src.tg, src.T, (int64_t)blockIdx.x * TILE,
                                 std::min<int64_t>((int64_t)(blockIdx.x + 1) * TILE, M) - 1);
    __syncthreads();
    const T *x = (const T *)src.x, *y = (const T *)src.y, *z = (const T *)src.z;
    const int dim = src.g.dim;
    const int64_t base = (int64_t)blockIdx.x * TILE;
    int bad = 0;
    // every coordinate load first, so that their latencies overlap
    T xc[kSrcItems][3];
#pragma unroll
    for (int r = 0; r < kSrcItems; ++r) {
        const int64_t jc =
            std::min<int64_t>(base + (int64_t)r * kSrcThreads + tid, (int64_t)M - 1);
        xc[r][0] = x[jc];
        xc[r][1] = dim >= 2 ? y[jc] : (T)0;
        xc[r][2] = dim == 3 ? z[jc] : (T)0;
    }
#pragma unroll
    for (int r = 0; r < kSrcItems; ++r) {
        const int64_t idx = base + (int64_t)r * kSrcThreads + tid;
        const bool valid = idx < M;
        uint32_t d = 0;
        if (valid) {
            T u[3];
            d = (point_key_of<T, BATCH>(src.g, xc[r], src.map, src.tg, src.T, nullptr, false,
                                        (int)idx, u, bad) >> shift) & dmask;
        }
        const uint32_t d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)d);
        const bool same = !valid || d == d0;
        if (__all(same)) {
            const uint64_t vm = __ballot(valid);
            if ((threadIdx.x & 63) == 0 && vm) atomicAdd(&h[d0], (uint32_t)__popcll(vm));
        } else if (valid) {
            atomicAdd(&h[d], 1u);
        }
    }
    if (bad) atomicOr(src.flag, 1);
    __syncthreads();
    store_counts(h, pitch, hist);
}

// Per-tile digit histogram, stored digit-major: hist[d * pitch + blk]; the
// digit is (key >> shift) & dmask with dmask + 1 <= 256.
template <int TILE>
__global__ void __launch_bounds__(kThreads)
k_radix_hist(const uint32_t *__restrict__ keys, int M, int shift, uint32_t dmask, int pitch,
             uint32_t *__restrict__ hist)
{
    constexpr int kItems = TILE / kThreads;
    __shared__ uint32_t h[256];
    const int tid = threadIdx.x;
    h[tid] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * TILE;
    // every key load first, so that their latencies overlap
    uint32_t kv[kItems];
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const int64_t idx = base + (int64_t)r * kThreads + tid;
        kv[r] = idx < M ? keys[idx] : 0u;
    }
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const int64_t idx = base + (int64_t)r * kThreads + tid;
        const bool valid = idx < M;
        const uint32_t d = valid ? (kv[r] >> shift) & dmask : 0u;
        // Lanes are contiguous in idx, so lane 0 is valid whenever any lane is.
        const uint32_t d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)d);
        const bool same = !valid || d == d0;
        if (__all(same)) {
            const uint64_t vm = __ballot(valid);
            if ((threadIdx.x & 63) == 0 && vm) atomicAdd(&h[d0], (uint32_t)__popcll(vm));
        } else if (valid) {
            atomicAdd(&h[d], 1u);
        }
    }
    __syncthreads();
    store_counts(h, pitch, hist);
}

// Stable scatter of one radix pass over a tile of TILE keys, with NT threads:
// wave w owns keys [blk*TILE + w*items*64, +items*64), items = TILE / NT, and
// walks them in rounds of 64 consecutive keys, so ranks grow with the input
// index.  Every array of the tile (key, value and ND payload planes of T, the
// bin-relative coordinates) is then rearranged in LDS into digit order and
// each digit's run written to its global range with consecutive threads on
// consecutive addresses.  Bound by latencies between its phases, not by
// bandwidth, so blocks have to overlap: all loads are issued before the
// ranking, and the arrays take turns in one stage of TILE values instead of
// filling the LDS together (one or two blocks a CU).  1e7 points in 2D 81 and
// 109 -> 80 and 78 us for the two passes, 1.7e7 in 3D 246 and 248 -> 170 and
// 240; 1024 threads with half the items each: 101 and 97, 205 and 231.
template <int TILE> constexpr int scatter_threads()
{
    return TILE < kTile ? 256 : (TILE == kTile ? 512 : 1024);
}

// SRC: 0 reads keys and payload; 1 computes them from the points (src, a
// plain plan); 2 the same for a batch (transform by binary search of pt_off).
// offs holds the scanned counts or, with `sums`, the counts themselves.
template <typename T, int ND, int SRC, int TILE, int NT = scatter_threads<TILE>()>
__global__ void __launch_bounds__(NT)
k_radix_scatter(const uint32_t *__restrict__ kin, const uint32_t *__restrict__ vin, int M,
                int shift, int dbits, int pitch, bool sums, const uint32_t *__restrict__ offs,
                uint32_t *__restrict__ kout, uint32_t *__restrict__ vout, Payload pl, KeySrc src)
{
    constexpr int kSWaves = NT / 64, kSItems = TILE / NT;
    __shared__ uint32_t cnt[kSWaves][256];   // running per-wave digit counts, then prefixes
    __shared__ uint32_t tstart[256];         // tile-local start of each digit run
    __shared__ uint32_t gbase[256];          // global start of each digit run
    __shared__ uint32_t wsum[4], asum[4];
    __shared__ __align__(16) unsigned char stage_raw[TILE * sizeof(T)];
    uint32_t *sU = reinterpret_cast<uint32_t *>(stage_raw);
    T *sT = reinterpret_cast<T *>(stage_raw);

    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    const int lane = tid & 63;
    for (int e = tid; e < kSWaves * 256; e += NT) (&cnt[0][0])[e] = 0;

    const int64_t tbase = (int64_t)blockIdx.x * TILE;
    const int64_t base = tbase + (int64_t)wave * (64 * kSItems);
    const int tcount = (int)std::min<int64_t>(TILE, (int64_t)M - tbase);
    if constexpr (SRC == 2)
        src.tg = tile_transforms(src.tg, src.T, tbase, tbase + tcount - 1);
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const uint32_t dmask = (1u << dbits) - 1u;
    uint32_t kk[kSItems], vv[kSItems], lp[kSItems];
    T pu[kSItems][ND];  // payload (SRC: the coordinates it is computed from, first)
    // every load first, so that their latencies overlap
    {
        const T *cs[3] = {(const T *)(SRC ? src.x : pl.in[0]), (const T *)(SRC ? src.y : pl.in[1]),
                          (const T *)(SRC ? src.z : pl.in[2])};
#pragma unroll
        for (int r = 0; r < kSItems; ++r) {
            const int64_t jc = std::min<int64_t>(base + r * 64 + lane, (int64_t)M - 1);
            if constexpr (!SRC) kk[r] = kin[jc];
            vv[r] = vin ? vin[jc] : (uint32_t)jc;
#pragma unroll
            for (int q = 0; q < ND; ++q) pu[r][q] = cs[q][jc];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSItems; ++r) {
        const int64_t idx = base + r * 64 + lane;
        const bool valid = idx < M;
        if constexpr (SRC) {
            kk[r] = 0u;
            if (valid) {
                T xc[3] = {pu[r][0], ND >= 2 ? pu[r][ND >= 2 ? 1 : 0] : (T)0,
                           ND == 3 ? pu[r][ND == 3 ? 2 : 0] : (T)0};
                T u[3];
                int bad = 0;
                kk[r] = point_key_of<T, SRC == 2>(src.g, xc, src.map, src.tg, src.T, nullptr,
                                                  false, (int)idx, u, bad);
#pragma unroll
                for (int q = 0; q < ND; ++q) pu[r][q] = u[q];
            }
        }
        const uint32_t d = (kk[r] >> shift) & dmask;
        uint64_t mask = __ballot(valid);
        for (int b = 0; b < dbits; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bb = __ballot(bit);
            mask &= bit ? bb : ~bb;
        }
        const uint32_t rank = (uint32_t)__popcll(mask & lt);
        uint32_t old = 0;
        if (valid) {
            old = cnt[wave][d];
            if (rank == 0) cnt[wave][d] = old + (uint32_t)__popcll(mask);
        }
        lp[r] = old + rank;  // within the wave's digit
    }
    __syncthreads();
    if (tid < 256) {
        // per digit: prefix over waves, then an exclusive scan over digits
        const int d = tid;
        uint32_t run = 0;
        for (int w = 0; w < kSWaves; ++w) {
            const uint32_t c = cnt[w][d];
            cnt[w][d] = run;
            run += c;
        }
        const uint32_t inc = wave_incl_scan(run, lane);
        uint32_t base_d = 0, all = 0;
        if (sums) {
            // this digit's points in earlier blocks, and in all of them
            const uint4 *row = reinterpret_cast<const uint4 *>(offs + (int64_t)d * pitch);
            const uint32_t me = blockIdx.x;
#pragma unroll 16
            for (uint32_t q = 0; q < (uint32_t)pitch / 4; ++q) {
                const uint4 v = row[q];
                base_d += (4 * q < me ? v.x : 0u) + (4 * q + 1 < me ? v.y : 0u) +
                          (4 * q + 2 < me ? v.z : 0u) + (4 * q + 3 < me ? v.w : 0u);
                all += v.x + v.y + v.z + v.w;
            }
        } else {
            base_d = offs[(int64_t)d * pitch + blockIdx.x];
        }
        const uint32_t ainc = wave_incl_scan(all, lane);
        if (lane == 63) {
            wsum[wave] = inc;
            asum[wave] = ainc;
        }
        tstart[d] = inc - run;  // within the wave's digits; completed below
        gbase[d] = base_d + (sums ? ainc - all : 0u);
    }
    __syncthreads();
    if (tid < 256) {
        for (int w = 0; w < wave; ++w) {
            tstart[tid] += wsum[w];
            gbase[tid] += sums ? asum[w] : 0u;
        }
    }
    __syncthreads();
    // position in the tile's digit order (none past the input's end)
#pragma unroll
    for (int r = 0; r < kSItems; ++r) {
        const uint32_t d = (kk[r] >> shift) & dmask;
        lp[r] += tstart[d] + cnt[wave][d];
        if (base + r * 64 + lane >= M || lp[r] >= (uint32_t)TILE) lp[r] = ~0u;
    }
    // each array in turn: scattered LDS writes, then contiguous runs to memory
    uint32_t gp[kSItems];
#pragma unroll
    for (int r = 0; r < kSItems; ++r)
        if (lp[r] != ~0u) sU[lp[r]] = kk[r];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSItems; ++k) {
        const int e = tid + k * NT;
        gp[k] = ~0u;
        if (e < tcount) {
            const uint32_t key = sU[e], d = (key >> shift) & dmask;
            gp[k] = gbase[d] + (uint32_t)e - tstart[d];
            if (gp[k] >= (uint32_t)M) gp[k] = ~0u;  // cannot happen when the counts agree
            else kout[gp[k]] = key;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSItems; ++r)
        if (lp[r] != ~0u) sU[lp[r]] = vv[r];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSItems; ++k)
        if (gp[k] != ~0u) vout[gp[k]] = sU[tid + k * NT];
#pragma unroll
    for (int q = 0; q < ND; ++q) {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSItems; ++r)
            if (lp[r] != ~0u) sT[lp[r]] = pu[r][q];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kSItems; ++k)
            if (gp[k] != ~0u) static_cast<T *>(pl.out[q])[gp[k]] = sT[tid + k * NT];
    }
}

// ---- generic exclusive scan (chunk totals; down-sweep adds earlier ones) ----
constexpr int kScanChunk = kThreads * kItems;

// Exclusive scan of one value per thread over the block; returns the block total.
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t &excl)
{
    __shared__ uint32_t wsum[kThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t inc = wave_incl_scan(v, lane);
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    uint32_t before = 0, total = 0;
    for (int w = 0; w < kThreads / 64; ++w) {
        if (w < wave) before += wsum[w];
        total += wsum[w];
    }
    __syncthreads();
    excl = before + inc - v;
    return total;
}

__global__ void __launch_bounds__(kThreads)
k_scan_reduce(const uint32_t *__restrict__ in, size_t n, uint32_t *__restrict__ partials)
{
    const size_t base = (size_t)blockIdx.x * kScanChunk;
    uint32_t s = 0;
    for (int r = 0; r < kItems; ++r) {
        const size_t i = base + (size_t)r * kThreads + threadIdx.x;
        if (i < n) s += in[i];
    }
    uint32_t ex;
    const uint32_t tot = block_excl_scan(s, ex);
    if (threadIdx.x == 0) partials[blockIdx.x] = tot;
}

__global__ void __launch_bounds__(kThreads)
k_scan_down(const uint32_t *__restrict__ in, uint32_t *__restrict__ out, size_t n,
            const uint32_t *__restrict__ partials)
{
    __shared__ uint32_t buf[kScanChunk + kScanChunk / 32];
    const size_t base = (size_t)blockIdx.x * kScanChunk;
    auto sk = [](int e) { return e + (e >> 5); };  // skew against bank conflicts
    for (int r = 0; r < kItems; ++r) {
        const int e = r * kThreads + threadIdx.x;
        const size_t i = base + e;
        buf[sk(e)] = (i < n) ? in[i] : 0u;
    }
    __syncthreads();
    // this chunk's offset: the sum of the earlier chunks' totals
    uint32_t before = 0;
    for (int k = threadIdx.x; k < (int)blockIdx.x; k += kThreads) before += partials[k];
    uint32_t ex0;
    before = block_excl_scan(before, ex0);
    uint32_t s = 0;
    for (int q = 0; q < kItems; ++q) s += buf[sk(threadIdx.x * kItems + q)];
    uint32_t ex;
    block_excl_scan(s, ex);
    uint32_t run = ex + before;
    for (int q = 0; q < kItems; ++q) {
        const int e = threadIdx.x * kItems + q;
        const uint32_t v = buf[sk(e)];
        buf[sk(e)] = run;
        run += v;
    }
    __syncthreads();
    for (int r = 0; r < kItems; ++r) {
        const int e = r * kThreads + threadIdx.x;
        const size_t i = base + e;
        if (i < n) out[i] = buf[sk(e)];
    }
}

// binstart[b] = first sorted position with key >= b: a wave per bin narrows
// the range 64-fold a step, four dependent loads for 1.6e7 points against 24
// of a binary search per thread (1e7 points in 4096 bins 12 -> 9 us, 1e5 in
// 256 bins 5.5 -> 3.8 us); above kWaveBins bins a thread per bin, which then
// fill the GPU.
constexpr int kWaveBins = 32768;
__global__ void __launch_bounds__(256)
k_binstart_wave(int M, int nbins, const uint32_t *__restrict__ skey,
                int32_t *__restrict__ binstart)
{
    const int b = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (b > nbins) return;
    int64_t lo = 0, hi = M;  // the answer lies in [lo, hi]
    while (lo < hi) {
        const int64_t len = hi - lo;
        // 64 probes, each the end of a sixty-fourth of [lo, hi), or all of it
        const auto probe = [&](int k) { return len <= 64 ? lo + k : lo + ((len * (k + 1)) >> 6) - 1; };
        const int64_t p = probe(lane);
        const bool below = p < hi && skey[p] < (uint32_t)b;
        const int n = (int)__popcll(__ballot(below));  // the first n probes are below
        if (len <= 64) {
            lo += n;
            break;
        }
        const int64_t nlo = n > 0 ? probe(n - 1) + 1 : lo;
        hi = n < 64 ? probe(n) : hi;
        lo = nlo;
    }
    if (lane == 0) binstart[b] = (int32_t)lo;
}

__global__ void k_binstart(int M, int nbins, const uint32_t *__restrict__ skey,
                           int32_t *__restrict__ binstart)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b > nbins) return;
    int lo = 0, hi = M;  // first position with skey >= b
    while (lo < hi) {
        const int mid = lo + ((hi - lo) >> 1);
        if (skey[mid] < (uint32_t)b) lo = mid + 1; else hi = mid;
    }
    binstart[b] = lo;
}

// msub of bin b: the plan's, or in a batch that of the bin's transform.
__device__ __forceinline__ int msub_of(int b, int msub, const TGeom *tg, const int32_t *bin_t)
{
    return tg ? tg[bin_t[b]].msub : msub;
}

__global__ void k_subcount(int nbins, int msub, const int32_t *__restrict__ binstart,
                           uint32_t *__restrict__ cnt, const TGeom *__restrict__ tg,
                           const int32_t *__restrict__ bin_t)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b > nbins) return;
    if (b == nbins) { cnt[b] = 0; return; }
    const int c = binstart[b + 1] - binstart[b];
    const int ms = msub_of(b, msub, tg, bin_t);
    cnt[b] = (uint32_t)((c + ms - 1) / ms);
}

// k_subcount and the scan of its counts in one block, for up to kScanBins bins
// (18225: 21 us, the separate launches about 10; 4096: 5.5 us); also clears
// the merge list's count.
constexpr int kScanBins = 8192;
__global__ void __launch_bounds__(1024)
k_subscan(int nbins, int msub, const int32_t *__restrict__ binstart, uint32_t *__restrict__ off,
          const TGeom *__restrict__ tg, const int32_t *__restrict__ bin_t,
          int32_t *__restrict__ nmerge)
{
    __shared__ uint32_t wsum[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (nmerge && tid == 0) *nmerge = 0;
    const int per = (nbins + 1023) / 1024, b0 = min(tid * per, nbins), b1 = min(b0 + per, nbins);
    const auto count = [&](int b) {
        const int c = binstart[b + 1] - binstart[b], ms = msub_of(b, msub, tg, bin_t);
        return (uint32_t)((c + ms - 1) / ms);
    };
    uint32_t mine = 0;
    for (int b = b0; b < b1; ++b) mine += count(b);
    const uint32_t inc = wave_incl_scan(mine, lane);
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    uint32_t run = inc - mine;
    for (int w = 0; w < wave; ++w) run += wsum[w];
    for (int b = b0; b < b1; ++b) {
        off[b] = run;
        run += count(b);
    }
    if (tid == 1023) off[nbins] = run;
}

// Subproblem records; with a merge list, also the leaders of tile groups to
// merge: subproblems q with (q - off[bin]) % G == 0 in bins with more than G
// of them (*nmerge is zero on entry).
__global__ void k_subfill(int nbins, int msub, int nsub_max, const int32_t *__restrict__ binstart,
                          const uint32_t *__restrict__ off, int32_t *__restrict__ sub,
                          int32_t *__restrict__ nsub, const TGeom *__restrict__ tg,
                          const int32_t *__restrict__ bin_t, int G,
                          int32_t *__restrict__ mergelist, int32_t *__restrict__ nmerge)
{
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    // the count is clamped to the list's capacity so that no consumer can
    // read past it, whatever the counts held
    const int total = std::min((int)off[nbins], nsub_max);
    if (q == 0) *nsub = total;
    if (q >= total || q >= nsub_max) return;
    int lo = 0, hi = nbins - 1;  // last bin b with off[b] <= q
    while (lo < hi) {
        const int mid = lo + ((hi - lo + 1) >> 1);
        if (off[mid] <= (uint32_t)q) lo = mid; else hi = mid - 1;
    }
    const int b = lo;
    const int ms = msub_of(b, msub, tg, bin_t);
    const int first = (int)off[b], s = q - first;
    const int start = binstart[b] + s * ms;
    const int len = std::min(ms, binstart[b + 1] - start);
    int4 rec;
    rec.x = b; rec.y = start; rec.z = len; rec.w = 0;
    reinterpret_cast<int4 *>(sub)[q] = rec;
    if (mergelist && (int)off[b + 1] - first > G && s % G == 0) mergelist[atomicAdd(nmerge, 1)] = q;
}

inline int nblocks(int64_t n, int t) { return (int)((n + t - 1) / t); }

}  // namespace

// (A plan's buffers serve smaller point sets too, and the count does not grow with
// M: 2^20 keys are 1024 small tiles, 2^20 + 1 are 257 large ones.)
size_t radix_hist_elems(int M)
{
    const int small = std::min(M, kSmallKeys);
    return (size_t)256 * std::max(hist_pitch(std::max(1, nblocks(small, tile_of(small)))),
                                  hist_pitch(std::max(1, nblocks(M, tile_of(M)))));
}

size_t scan_partial_elems(size_t n) { return (n + kScanChunk - 1) / kScanChunk + 1; }

hipError_t scan_exclusive(const uint32_t *in, uint32_t *out, size_t n, uint32_t *partials,
                          hipStream_t s)
{
    if (n == 0) return hipSuccess;
    const int np = (int)((n + kScanChunk - 1) / kScanChunk);
    // chunk totals, then each chunk adds the totals before it (one chunk:
    // nothing before it, so the first kernel is skipped)
    if (np > 1)
        hipLaunchKernelGGL(k_scan_reduce, dim3(np), dim3(kThreads), 0, s, in, n, partials);
    hipLaunchKernelGGL(k_scan_down, dim3(np), dim3(kThreads), 0, s, in, out, n,
                       (const uint32_t *)partials);
    return hipGetLastError();
}

hipError_t launch_binkey(const Geom &g, int prec, int M, const void *x, const void *y,
                         const void *z, uint32_t *key, void *const u_in[3], int *flag,
                         hipStream_t s, const TGeom *tg, int T, const PtMap *map)
{
    if (M == 0) return hipSuccess;
    const dim3 grid(nblocks(M, kThreads)), blk(kThreads);
    PtMap pm{};
    if (map) pm = *map;
#define MN_BK(TT, BB)                                                                        \
    hipLaunchKernelGGL((k_binkey<TT, BB>), grid, blk, 0, s, g, M, (const TT *)x, (const TT *)y, \
                       (const TT *)z, key, (TT *)u_in[0], (TT *)u_in[1], (TT *)u_in[2], flag, tg, T, \
                       pm)
    if (prec == 0) {
        if (tg) MN_BK(float, true); else MN_BK(float, false);
    } else {
        if (tg) MN_BK(double, true); else MN_BK(double, false);
    }
#undef MN_BK
    return hipGetLastError();
}

int radix_passes(int bits) { return std::max(1, (bits + 7) / 8); }

hipError_t radix_sort(int M, int bits, int prec, int dim, uint32_t *keysA, uint32_t *valsA,
                      uint32_t *keysB, uint32_t *valsB, const Payload *pays, uint32_t *hist,
                      size_t hist_elems, uint32_t *partials, uint32_t **keys_out, uint32_t **vals_out, hipStream_t s,
                      const KeySrc *src)
{
    // Keys start in keysA with implicit values 0..M-1; each pass moves the
    // pairs to the other buffer.  Pass p moves the payload as pays[p] says.
    // Digits of equal width dbits <= 8 over the passes: fewer digits per pass
    // mean longer runs of each digit per tile, hence more coalesced writes.
    const int passes = radix_passes(bits);
    const int dbits = std::max(1, (bits + passes - 1) / passes);
    const uint32_t dmask = (1u << dbits) - 1u;
    uint32_t *kb[2] = {keysA, keysB}, *vb[2] = {valsA, valsB};
    int cur = 0;
    for (int p = 0; p < passes; ++p) {
        if (M > 0) {
            const int shift = dbits * p;
            // pass 0 from the points themselves when a source is given
            const int from = (p == 0 && src) ? (src->tg ? 2 : 1) : 0;
            const int tile = tile_of(M, !from && dim == 3 && prec == 0);
            const int nblk = std::max(1, nblocks(M, tile)), pitch = hist_pitch(nblk);
            if ((size_t)256 * pitch > hist_elems) return hipErrorInvalidValue;
            const bool sums = nblk <= kFusedBlocks;  // the scatter sums the counts itself
            const KeySrc ks = src ? *src : KeySrc{};
            const uint32_t *vin = p == 0 ? nullptr : (const uint32_t *)vb[cur];
            const auto pass = [&](auto tag) -> hipError_t {
                constexpr int TILE = decltype(tag)::value;
#define MN_HSRC(TT, BB)                                                                       \
    hipLaunchKernelGGL((k_radix_hist_src<TT, BB, TILE>), dim3(nblk), dim3(kSrcThreads), 0, s,  \
                       ks, M, shift, dmask, pitch, hist)
                constexpr bool wide = TILE == kTileWide;
                if (from == 0 || wide)
                    hipLaunchKernelGGL((k_radix_hist<TILE>), dim3(nblk), dim3(kThreads), 0, s,
                                       (const uint32_t *)kb[cur], M, shift, dmask, pitch, hist);
                if constexpr (!wide) {
                    if (from == 2) {
                        if (prec == 0) MN_HSRC(float, true);
                        else MN_HSRC(double, true);
                    } else if (from == 1) {
                        if (prec == 0) MN_HSRC(float, false);
                        else MN_HSRC(double, false);
                    }
                }
#undef MN_HSRC
                // digits above dmask are empty: only the first dmask + 1 rows are scanned
                if (!sums) {
                    const hipError_t e =
                        scan_exclusive(hist, hist, (size_t)(dmask + 1) * pitch, partials, s);
                    if (e != hipSuccess) return e;
                }
#define MN_SCATTER1(TT, DD, SS)                                                             \
    do {                                                                                    \
        hipLaunchKernelGGL((k_radix_scatter<TT, DD, SS, TILE>), dim3(nblk),                 \
                           dim3(scatter_threads<TILE>()), 0, s,                             \
                           (const uint32_t *)kb[cur], vin, M, shift, dbits, pitch, sums,    \
                           (const uint32_t *)hist, kb[1 - cur], vb[1 - cur], pays[p], ks);  \
    } while (0)
#define MN_SCATTER(TT, DD)                                                                  \
    do {                                                                                    \
        if (from == 2) MN_SCATTER1(TT, DD, 2);                                              \
        else if (from == 1) MN_SCATTER1(TT, DD, 1);                                         \
        else MN_SCATTER1(TT, DD, 0);                                                        \
    } while (0)
                if constexpr (wide) {
                    MN_SCATTER1(float, 3, 0);
                } else if (prec == 0) {
                    if (dim == 1) MN_SCATTER(float, 1);
                    else if (dim == 2) MN_SCATTER(float, 2);
                    else MN_SCATTER(float, 3);
                } else {
                    if (dim == 1) MN_SCATTER(double, 1);
                    else if (dim == 2) MN_SCATTER(double, 2);
                    else MN_SCATTER(double, 3);
                }
#undef MN_SCATTER
#undef MN_SCATTER1
                return hipSuccess;
            };
            const hipError_t e =
                tile == kTileWide ? pass(std::integral_constant<int, kTileWide>())
                : tile == kTile   ? pass(std::integral_constant<int, kTile>())
                                  : pass(std::integral_constant<int, kTileSmall>());
            if (e != hipSuccess) return e;
        }
        cur = 1 - cur;
    }
    *keys_out = kb[cur];
    *vals_out = vb[cur];
    return hipGetLastError();
}

hipError_t launch_binstart(int M, int nbins, const uint32_t *skey, int32_t *binstart,
                           hipStream_t s)
{
    if (nbins <= kWaveBins)
        hipLaunchKernelGGL(k_binstart_wave, dim3(nblocks(nbins + 1, 4)), dim3(256), 0, s, M,
                           nbins, skey, binstart);
    else
        hipLaunchKernelGGL(k_binstart, dim3(nblocks(nbins + 1, 256)), dim3(256), 0, s, M, nbins,
                           skey, binstart);
    return hipGetLastError();
}

// ---- processing order of the SM kernels -----------------------------------
// The SM kernels give each lane of a wave one point and have all lanes touch
// the same tap of their points at once, so a wave's LDS addresses are the
// points' tile start cells plus a common offset.  The LDS serves 64-bit
// accesses sixteen lanes at a time and stalls when two of them hit the same
// bank; the banks follow the cell index modulo 16 (two or four banks per
// cell), so sixteen points whose start-cell indices differ modulo 16 are
// served without conflict whatever the tap.  This kernel orders each
// subproblem's points round-robin over their start-cell index modulo 16:
// every point of rank k in its residue class comes before every point of
// rank k + 1, residues ascending within a rank, i.e. point (r, k) goes to
//   pos = sum_t min(c_t, k) + #{t < r : c_t > k}     (c_t = class sizes).
// The sorted coordinates, the permutation, each point's sorted position and
// its slot in the spreading kernels' start-cell histogram are written in
// that order.  Subproblems above kBalCap points keep their sorted order.
// A block loads a subproblem's points once (coalesced, kBalItems per
// thread), ranks them in their classes with LDS atomics, then writes each
// output array through an LDS stage so that the global stores are
// contiguous too.  The ranks come from LDS atomics, so the order within a
// class may differ between runs; the SM kernels' results do not depend on
// the order (integer tile sums, per-point interpolation).
constexpr int kBalCap = 4096;
constexpr int kBalThreads = 256;
// Two instantiations share the subproblems: ITEMS = 8 takes those of up to
// 2048 points (3D bins, typically), ITEMS = 16 the rest, so small
// subproblems neither load unused rounds nor hold the larger one's registers.
template <typename T, int DIM, int ITEMS>
__global__ void __launch_bounds__(kBalThreads)
k_balance(Geom g, const int32_t *__restrict__ sub, const int32_t *__restrict__ nsubp,
          const T *__restrict__ u0, const T *__restrict__ u1, const T *__restrict__ u2,
          const int32_t *__restrict__ perm, T *__restrict__ v0, T *__restrict__ v1,
          T *__restrict__ v2, int32_t *__restrict__ vperm, int32_t *__restrict__ spos,
          uint16_t *__restrict__ hslot)
{
    constexpr int kBalItems = ITEMS;
    constexpr int kLo = ITEMS == 8 ? 0 : 8 * kBalThreads;         // sizes n with kLo < n
    constexpr int kHi = ITEMS == 8 ? 8 * kBalThreads : 1 << 30;   // and n <= kHi
    __shared__ unsigned cnt[16];
    __shared__ __align__(16) unsigned char stage_raw[kBalItems * kBalThreads * sizeof(T)];
    T *sT = reinterpret_cast<T *>(stage_raw);
    int32_t *sI = reinterpret_cast<int32_t *>(stage_raw);
    uint16_t *sH = reinterpret_cast<uint16_t *>(stage_raw);
    const int tid = threadIdx.x;
    const int P = (g.w + 1) / 2;
    const int p1 = g.m[0] + 2 * P, p2 = g.m[1] + 2 * P;
    const T lead = (T)P - (T)(0.5 * g.w);
    const StartHist hg = start_hist_rt(DIM, g.w, g.m[0], g.m[1], g.m[2]);
    // the spreading kernels' start-cell histogram slot (same expressions)
    const auto slot = [&](T a, T b, T c) {
        return (uint16_t)hist_slot_rt(hg, DIM >= 2 ? start_cell_rt<T>(b, g.w) : 0,
                                      DIM == 3 ? start_cell_rt<T>(c, g.w) : 0,
                                      start_cell_rt<T>(a, g.w));
    };
    const int nsub = *nsubp;
    for (int q = blockIdx.x; q < nsub; q += gridDim.x) {
        const int4 rec = reinterpret_cast<const int4 *>(sub)[q];
        const int n = rec.z;
        if (n <= kLo || n > kHi) continue;  // the other instantiation's subproblem
        if (n > kBalCap) {  // the same for the whole block: keep the sorted order
            for (int j = tid; j < n; j += kBalThreads) {
                const int i = rec.y + j;
                const T a = u0[i], b = DIM >= 2 ? u1[i] : (T)0, c = DIM == 3 ? u2[i] : (T)0;
                v0[i] = a;
                if (DIM >= 2) v1[i] = b;
                if (DIM == 3) v2[i] = c;
                vperm[i] = perm[i];
                spos[i] = i;
                hslot[i] = slot(a, b, c);
            }
            continue;
        }
        if (tid < 16) cnt[tid] = 0u;
        __syncthreads();
        T a[kBalItems], b[kBalItems], c[kBalItems];
        int pm[kBalItems], pos[kBalItems];
#pragma unroll
        for (int it = 0; it < kBalItems; ++it) {
            const int j = tid + it * kBalThreads;
            const int i = rec.y + min(j, n - 1);
            a[it] = u0[i];
            b[it] = DIM >= 2 ? u1[i] : (T)0;
            c[it] = DIM == 3 ? u2[i] : (T)0;
            pm[it] = perm[i];
        }
#pragma unroll
        for (int it = 0; it < kBalItems; ++it) {
            const int j = tid + it * kBalThreads;
            pos[it] = 0;
            if (j < n) {
                int base = (int)ceil(a[it] + lead);
                if (DIM >= 2) base += p1 * (int)ceil(b[it] + lead);
                if (DIM == 3) base += p1 * p2 * (int)ceil(c[it] + lead);
                const unsigned r = (unsigned)base & 15u;
                pos[it] = (int)(r | (atomicAdd(&cnt[r], 1u) << 4));
            }
        }
        __syncthreads();
        unsigned cc[16];
#pragma unroll
        for (int t = 0; t < 16; ++t) cc[t] = cnt[t];
#pragma unroll
        for (int it = 0; it < kBalItems; ++it) {
            const unsigned r = (unsigned)pos[it] & 15u, k = (unsigned)pos[it] >> 4;
            int o = 0;
#pragma unroll
            for (int t = 0; t < 16; ++t) o += (int)min(cc[t], k) + ((t < (int)r && cc[t] > k) ? 1 : 0);
            pos[it] = o;
        }
        // each output through the stage: scattered LDS writes, contiguous stores
        const auto emit = [&](auto *stage, auto *dst, auto value) {
#pragma unroll
            for (int it = 0; it < kBalItems; ++it)
                if (tid + it * kBalThreads < n) stage[pos[it]] = value(it);
            __syncthreads();
            for (int j = tid; j < n; j += kBalThreads) dst[rec.y + j] = stage[j];
            __syncthreads();
        };
        emit(sT, v0, [&](int it) { return a[it]; });
        if constexpr (DIM >= 2) emit(sT, v1, [&](int it) { return b[it]; });
        if constexpr (DIM == 3) emit(sT, v2, [&](int it) { return c[it]; });
        emit(sI, vperm, [&](int it) { return pm[it]; });
        emit(sI, spos, [&](int it) { return rec.y + tid + it * kBalThreads; });
        emit(sH, hslot, [&](int it) { return slot(a[it], b[it], c[it]); });
    }
}

// Processing order of the matrix-core kernels (mfma_kernels.h): the points of
// a subproblem by window group, groups in x-fastest order, points of a group
// in sorted order.  A group is the start cells (start / s) per dimension.  A
// stable counting sort: each wave ranks a contiguous share of the points by
// ballots over the group's bits, so the order (and the sums that follow it)
// is the same in every run.  Bound by its traffic, as k_balance is.
constexpr int kGroupMax = 256;
template <typename T, int DIM, int ITEMS>
__global__ void __launch_bounds__(kBalThreads)
k_group(Geom g, int s, int3 ng, int bits, const int32_t *__restrict__ sub,
        const int32_t *__restrict__ nsubp, const T *__restrict__ u0, const T *__restrict__ u1,
        const T *__restrict__ u2, const int32_t *__restrict__ perm, T *__restrict__ v0,
        T *__restrict__ v1, T *__restrict__ v2, int32_t *__restrict__ vperm,
        int32_t *__restrict__ spos)
{
    constexpr int kLo = ITEMS == 8 ? 0 : 8 * kBalThreads;
    constexpr int kHi = ITEMS == 8 ? 8 * kBalThreads : 16 * kBalThreads;
    constexpr int kWaves = kBalThreads / 64;
    __shared__ uint32_t cnt[kWaves][kGroupMax];
    __shared__ uint32_t first[kGroupMax];
    __shared__ __align__(16) unsigned char stage_raw[ITEMS * kBalThreads * sizeof(T)];
    T *sT = reinterpret_cast<T *>(stage_raw);
    int32_t *sI = reinterpret_cast<int32_t *>(stage_raw);
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    const int nsub = *nsubp;
    for (int q = blockIdx.x; q < nsub; q += gridDim.x) {
        const int4 rec = reinterpret_cast<const int4 *>(sub)[q];
        const int n = rec.z;
        if (n <= kLo || n > kHi) continue;  // the other instantiation's subproblem
        for (int e = tid; e < kWaves * kGroupMax; e += kBalThreads) (&cnt[0][0])[e] = 0u;
        __syncthreads();
        // wave w takes points w share .. (w + 1) share, 64 at a time
        const int share = (n + kBalThreads - 1) / kBalThreads * 64;
        T a[ITEMS], b[ITEMS], c[ITEMS];
        int pm[ITEMS], pos[ITEMS], grp[ITEMS];
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const int i = rec.y + min(wave * share + it * 64 + lane, n - 1);
            a[it] = u0[i];
            b[it] = DIM >= 2 ? u1[i] : (T)0;
            c[it] = DIM == 3 ? u2[i] : (T)0;
            pm[it] = perm[i];
        }
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const int j = wave * share + it * 64 + lane;
            const bool valid = it * 64 < share && j < n;
            int gr = start_cell_rt<T>(a[it], g.w) / s;
            if (DIM >= 2) gr += ng.x * (start_cell_rt<T>(b[it], g.w) / s);
            if (DIM == 3) gr += ng.x * ng.y * (start_cell_rt<T>(c[it], g.w) / s);
            gr = min(max(gr, 0), kGroupMax - 1);
            uint64_t mask = __ballot(valid);
            for (int k = 0; k < bits; ++k) {
                const bool bit = (gr >> k) & 1;
                const uint64_t bb = __ballot(bit);
                mask &= bit ? bb : ~bb;
            }
            const uint32_t rank = (uint32_t)__popcll(mask & lt);
            uint32_t old = 0;
            if (valid) {
                old = cnt[wave][gr];
                if (rank == 0) cnt[wave][gr] = old + (uint32_t)__popcll(mask);
            }
            grp[it] = gr;
            pos[it] = (int)(old + rank);
        }
        __syncthreads();
        if (tid < kGroupMax) {  // (kBalThreads == kGroupMax)
            uint32_t run = 0;
            for (int w = 0; w < kWaves; ++w) {
                const uint32_t t = cnt[w][tid];
                cnt[w][tid] = run;
                run += t;
            }
            uint32_t ex;
            block_excl_scan(run, ex);
            first[tid] = ex;
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) pos[it] += (int)(first[grp[it]] + cnt[wave][grp[it]]);
        const auto emit = [&](auto *stage, auto *dst, auto value) {
#pragma unroll
            for (int it = 0; it < ITEMS; ++it)
                if (it * 64 < share && wave * share + it * 64 + lane < n) stage[pos[it]] = value(it);
            __syncthreads();
            for (int j = tid; j < n; j += kBalThreads) dst[rec.y + j] = stage[j];
            __syncthreads();
        };
        emit(sT, v0, [&](int it) { return a[it]; });
        if constexpr (DIM >= 2) emit(sT, v1, [&](int it) { return b[it]; });
        if constexpr (DIM == 3) emit(sT, v2, [&](int it) { return c[it]; });
        emit(sI, vperm, [&](int it) { return pm[it]; });
        emit(sI, spos, [&](int it) { return rec.y + wave * share + it * 64 + lane; });
    }
}

namespace {
__global__ void k_iota(int n, int32_t *__restrict__ out)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
        out[i] = i;
}
}  // namespace

hipError_t launch_iota(int32_t *out, int n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_iota, dim3(std::min(nblocks(n, 256), 4096)), dim3(256), 0, s, n, out);
    return hipGetLastError();
}

hipError_t launch_balance(const Geom &g, int prec, int nsub_max, int msub, const int32_t *sub,
                          const int32_t *nsub, const void *const u[3], const int32_t *perm,
                          void *const v[3], int32_t *vperm, int32_t *spos, uint16_t *hslot,
                          hipStream_t s)
{
    if (nsub_max <= 0) return hipSuccess;
    const dim3 grid(std::max(1, std::min(nsub_max, 256 * 8)));
#define MN_BAL1(TT, DD, II)                                                                    \
    hipLaunchKernelGGL((k_balance<TT, DD, II>), grid, dim3(kBalThreads), 0, s, g, sub, nsub,   \
                       (const TT *)u[0], (const TT *)u[1], (const TT *)u[2], perm, (TT *)v[0],  \
                       (TT *)v[1], (TT *)v[2], vperm, spos, hslot)
#define MN_BAL(TT, DD)                                                                         \
    do {                                                                                       \
        MN_BAL1(TT, DD, 8);                                                                    \
        if (msub > 8 * kBalThreads) MN_BAL1(TT, DD, 16);                                       \
    } while (0)
    if (prec == 0) {
        if (g.dim == 1) MN_BAL(float, 1);
        else if (g.dim == 2) MN_BAL(float, 2);
        else MN_BAL(float, 3);
    } else {
        if (g.dim == 1) MN_BAL(double, 1);
        else if (g.dim == 2) MN_BAL(double, 2);
        else MN_BAL(double, 3);
    }
#undef MN_BAL
#undef MN_BAL1
    return hipGetLastError();
}

hipError_t launch_group(const Geom &g, int prec, int span, int nsub_max, const int32_t *sub,
                        const int32_t *nsub, const void *const u[3], const int32_t *perm,
                        void *const v[3], int32_t *vperm, int32_t *spos, hipStream_t st)
{
    if (nsub_max <= 0) return hipSuccess;
    int ng[3];
    int total = 1, bits = 0;
    for (int d = 0; d < 3; ++d) {
        ng[d] = d < g.dim ? (g.m[d] + 1) / span + 1 : 1;  // start cells 0 .. m + 1
        total *= ng[d];
    }
    if (total > kGroupMax || g.dim != 3 || prec == 0) return hipErrorInvalidValue;
    while ((1 << bits) < total) ++bits;
    const dim3 grid(std::max(1, std::min(nsub_max, 256 * 8)));
#define MN_GRP(II)                                                                           \
    hipLaunchKernelGGL((k_group<double, 3, II>), grid, dim3(kBalThreads), 0, st, g, span,    \
                       make_int3(ng[0], ng[1], ng[2]), bits, sub, nsub, (const double *)u[0], \
                       (const double *)u[1], (const double *)u[2], perm, (double *)v[0],     \
                       (double *)v[1], (double *)v[2], vperm, spos)
    MN_GRP(8);
    MN_GRP(16);
#undef MN_GRP
    return hipGetLastError();
}

hipError_t launch_subproblems(int nbins, int msub, int nsub_max, const int32_t *binstart,
                              int32_t *subcount, uint32_t *partials, int32_t *sub,
                              int32_t *nsub, int G, int32_t *mergelist, int32_t *nmerge,
                              hipStream_t s, const TGeom *tg, int T, const int32_t *bin_t)
{
    if (tg && !bin_t) return hipErrorInvalidValue;
    (void)T;
    uint32_t *cnt = reinterpret_cast<uint32_t *>(subcount);
    if (nbins <= kScanBins) {
        hipLaunchKernelGGL(k_subscan, dim3(1), dim3(1024), 0, s, nbins, msub, binstart, cnt, tg,
                           bin_t, nmerge);
    } else {
        if (nmerge) {
            const hipError_t e = launch_zero(nmerge, 4, s);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(k_subcount, dim3(nblocks(nbins + 1, 256)), dim3(256), 0, s, nbins,
                           msub, binstart, cnt, tg, bin_t);
        const hipError_t e = scan_exclusive(cnt, cnt, (size_t)nbins + 1, partials, s);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_subfill, dim3(nblocks(std::max(nsub_max, 1), 256)), dim3(256), 0, s,
                       nbins, msub, nsub_max, binstart, (const uint32_t *)cnt, sub, nsub, tg,
                       bin_t, G, mergelist, nmerge);
    return hipGetLastError();
}

}  // namespace mn
