// Host-side helpers shared by plans and batches of libmnufft (not public).
#pragma once

#include "../../include/mnufft.h"
#include "internal.h"

#include <stdint.h>
#include <functional>
#include <utility>
#include <vector>

namespace mn {
namespace host {

constexpr double kPi = 3.141592653589793;

// Kernel width w = ceil(log10(1/eps)) + 1 (Sec. II); a guard of 1e-9 keeps
// decade tolerances (whose logarithm is not exactly an integer in floating
// point) on the intended side.
int width_for_eps(double eps);

// Smallest 2^a 3^b 5^c >= max(2N, 2w) (Sec. II).
// General upsampling factor sigma (sigma = 2: the rule above, exactly).
int width_for_eps_sigma(double eps, double sigma);
double beta_for(int w, double sigma);
int64_t fine_size(int64_t N, int w, double sigma = 2.0);

// p_k = (2/w) / phi_hat(alpha k) * (-1)^k for k in I_N, alpha = w pi / n
// (Sec. II-A step 3; the sign is the lattice phase of grid point l at l h - pi).
void correction(int64_t N, int64_t n, int w, double beta, std::vector<double> &p);

// phi_hat(xi) = int_{-1}^{1} phi_beta(z) cos(xi z) dz at every xi (tanh-sinh
// quadrature, 513 nodes).
void es_fourier(double beta, const std::vector<double> &xi, std::vector<double> &out);

// Whether single precision rounding on the fine grid reaches the results
// amplified more than 200 times: by the rms of the correction factors over
// the band, which are far above one for wide kernels at upsampling factors
// near 1.25 (3D, eps 1e-6, sigma = 1.25: 1550 times, results 2.2e-5 from the
// sums, all of it such rounding).  There any other FFT or order of sums gives
// other noise of the same size (3.3e-5 between two), rocFFT's a little less
// than the own passes' (2.2e-5 against 2.5e-5): such plans keep rocFFT.
// (Single precision below sigma = 2 also keeps msub and a batch's own bins:
// the spreading quantum follows the subproblems and is amplified likewise.)
bool noisy_factors(int prec, int w, double beta, double sigma, int dim);

// Default bin extents for a fine grid n (dim dimensions): 64 cells in 1D,
// 32 x 32 in 2D and 16 x 8 x 8 in 3D (measured on gfx950; the paper's V100
// choice was 32 x 32 and 16 x 16 x 2, Sec. III-A, first remark), each at most
// the grid, then halved along the longest side while the grid holds fewer
// than kMinBins bins and that side is above kMinSide: a small grid cut into
// few bins leaves most of the GPU's compute units idle.
constexpr int64_t kMinBins = 1024;
constexpr int kMinSide = 8;
void default_bins(int dim, const int64_t n[3], int m[3]);

// Give a type 1 / 2 plan another method, bins and msub (c.method, binsize,
// msub; the rest of c is ignored), keeping its fine grid, FFT and correction
// factors; the points must be set again.  Used by the autotuner to time
// candidates on one plan.  Errors: ERR_ARG (bins that do not fit LDS for
// method SM, a type 3 plan), ERR_ALLOC, ERR_HIP.
int plan_set_params(mnufft_plan p, const mnufft_opts &c);

// Bits needed to hold bin indices 0 .. nbins - 1.
int bits_for(int64_t nbins);

// Cover table of the SM add-back for one dimension: for every grid index l,
// the (bin, offset in its padded tile) pairs whose tile lands on l after
// periodic wrapping; rows padded to the largest count kmax with bin -1.
void cover_table(int n, int m, int B, int P, std::vector<int2> &tab, int &kmax);

// Device memory from and to the pool (pool.cpp), on the current device.  `idle`:
// the device is known not to use the block any more; others are freed, which
// waits for their users.
hipError_t pool_alloc(void **ptr, size_t bytes);
void pool_free(void *ptr, bool idle);

// Where the work on an owner's buffers may still be pending: on its stream, or,
// when a call was captured there (a graph may be replayed anywhere) or the
// stream has been changed, on any stream of its device.
struct InUse {
    int device = -1;         // the owner's
    bool elsewhere = false;
    // To be called before work is enqueued on s.
    void note(hipStream_t s);
    // Waits for that work; false when it could not.
    bool wait(hipStream_t s) const;
};

// Per-stage HIP-event timers on one stream.
struct Timers {
    bool on = false;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> ev[MNUFFT_NSTAGES];
    size_t used[MNUFFT_NSTAGES] = {};
    // Sum of recorded durations per stage (synchronises s); optionally clears.
    int read(hipStream_t s, double *ms, int64_t *count, int reset);
    void destroy();
};

// Brackets one stage with an event pair when the timers are on.
struct StageTimer {
    Timers &t;
    int stage;
    hipStream_t s;
    bool on;
    StageTimer(Timers &tt, int st, hipStream_t ss);
    ~StageTimer();
};

// Fine-grid FFT with truncation / zero padding and correction factors in its
// passes.  `ok` is false when a dimension is too long for a block's LDS (or a
// line's pass for its threads): those grids use rocFFT and the correction
// kernels.
enum FftBuf { kFftGrid = 0, kFftModes = 1, kFftWork = 2 };
using FftAlloc = std::function<int(void **, size_t)>;
struct FftStep {
    FftPass p;
    int V = 16, form = 0, src = 0, dst = 0;
    bool rotate = false;  // takes the two-step table of a long line
    long long tiles = 0;
};
struct FftPlan {
    bool ok = false;
    int prec = 0;
    std::vector<FftStep> dir[2];   // type 1, type 2
    int64_t work_cells = 0;        // workspace of type 2 (1D, two-pass), complex values
    // Tables are allocated with `alloc` and filled on s (the caller waits).
    int make(int dim, const int64_t *N, const int *n, int64_t nt, int prec_,
             const void *const pf[3], const FftAlloc &alloc, hipStream_t s);
    // type 1: grid (overwritten) -> modes; type 2: modes -> grid.
    int run(int type, int sign, void *grid, void *modes, void *work, hipStream_t s) const;
};
// The same for every transform of a batch (2D / 3D), one launch per pass.
struct FftBatch {
    bool ok = false;
    int prec = 0, steps = 0, ntab = 0;
    const FftPass *table[3] = {};
    int form[3] = {}, src[3] = {}, dst[3] = {}, threads[3] = {}, lds[3] = {};
    long long tiles[3] = {};
    int make(int type, int dim, int iflag, const std::vector<TGeom> &geo, int prec_,
             const void *const pf[3], const FftAlloc &alloc, hipStream_t s);
    int run(void *grid, void *modes, hipStream_t s) const;
};

// In-place C2C rocFFT plan of the given lengths (first fastest); `sign` is
// the exponent sign.  Returns MNUFFT_OK or MNUFFT_ERR_FFT; *work receives the
// work-buffer size.
int make_rocfft(int prec, int dim, const int *n, size_t batch, int sign, void **plan,
                size_t *work);

}  // namespace host
}  // namespace mn
