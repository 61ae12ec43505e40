// Host side of the fine-grid FFT: which lines each pass of a plan or batch
// transforms, and where they come from and go to (kernels in fft_kernels.h).
#include "host_common.h"

#include <algorithm>
#include <cmath>

namespace mn {
namespace host {
namespace {

// Longest 1D transform done as one pass; above it, a pass over columns and
// one over rows (a single line would occupy one compute unit).
constexpr int64_t kOneLine = 4096;

struct Pass {
    FftPass p{};
    int src, dst;    // FftBuf
    int64_t nt;      // transforms
    int form = 0;
    bool rows;
    bool rotate = false;  // scales its outputs by FftPass::tw4
};

FftPass blank()
{
    FftPass p{};
    p.nb = 1;
    p.pe = 1;
    return p;
}

// The passes of one direction: type 1 (grid -> modes) or type 2 (modes ->
// grid) of a dim-dimensional grid n with N kept modes per dimension.
void passes_of(int type, int dim, const int64_t *N, const int *n, int64_t nt,
               const void *const pf[3], int64_t goff, int64_t moff, int fourA,
               std::vector<Pass> &out)
{
    const int64_t n1 = n[0], n2 = dim >= 2 ? n[1] : 1, n3 = dim == 3 ? n[2] : 1;
    const int64_t N1 = N[0], N2 = dim >= 2 ? N[1] : 1, N3 = dim == 3 ? N[2] : 1;
    const int64_t cells = n1 * n2 * n3, modes = N1 * N2 * N3;
    const bool t1 = type == 1;
    // grid side (g_*) and mode side (m_*) of a pass that truncates or pads
    const auto ends = [&](Pass &q, int64_t ge, int64_t ga, int64_t gb, int64_t gt, int64_t me,
                          int64_t ma, int64_t mb, int64_t mt, int64_t keep, bool user) {
        FftPass &p = q.p;
        p.cut = (int)keep;
        q.form = t1 ? 1 : 2;
        p.s_e = t1 ? ge : me; p.s_a = t1 ? ga : ma; p.s_b = t1 ? gb : mb; p.s_t = t1 ? gt : mt;
        p.d_e = t1 ? me : ge; p.d_a = t1 ? ma : ga; p.d_b = t1 ? mb : gb; p.d_t = t1 ? mt : gt;
        const int64_t mo = user ? moff : goff;
        p.s0 = t1 ? goff : mo;
        p.d0 = t1 ? mo : goff;
        q.src = t1 || !user ? kFftGrid : kFftModes;
        q.dst = t1 && user ? kFftModes : kFftGrid;
    };
    if (dim == 1 && !fourA) {
        Pass q;
        q.p = blank();
        q.nt = 1;
        q.rows = true;
        q.p.n = q.p.full = (int)n1;
        q.p.na = (int)nt;
        ends(q, 1, n1, 0, 0, 1, N1, 0, 0, N1, true);
        q.p.scale = 1;
        q.p.fe = pf[0];
        out.push_back(q);
        return;
    }
    if (dim == 1) {
        // l = la B + lb: columns of length A, a rotation, rows of length B;
        // frequency ka + A kb leaves row ka at kb
        const int A = fourA, B = (int)(n1 / fourA);
        Pass c, r;
        c.p = r.p = blank();
        c.nt = r.nt = nt;
        c.rows = r.rows = false;
        c.p.n = A;
        c.p.na = B;
        r.p.n = B;
        r.p.na = A;
        c.p.full = r.p.full = (int)n1;
        c.p.col0 = c.p.col1 = 1;
        r.p.col0 = 0;
        r.p.col1 = 1;
        c.rotate = true;
        c.p.s_e = c.p.d_e = B;
        c.p.s_a = c.p.d_a = 1;
        c.p.s_t = c.p.d_t = n1;
        r.p.s_e = 1;
        r.p.s_a = B;
        r.p.s_t = n1;
        r.p.pe = A;
        r.p.pa = 1;
        if (t1) {
            c.src = c.dst = r.src = kFftGrid;
            r.dst = kFftModes;
            r.p.cut = (int)N1;
            r.form = 1;
            r.p.d_e = 1;
            r.p.d_t = N1;
            r.p.scale = 1;
            r.p.fe = pf[0];
        } else {
            c.src = kFftModes;
            c.dst = r.src = kFftWork;
            r.dst = kFftGrid;
            c.p.cut = (int)N1;
            c.form = 2;
            c.p.pe = B;
            c.p.pa = 1;
            c.p.s_e = 1;
            c.p.s_a = 0;
            c.p.s_t = N1;
            c.p.scale = 1;
            c.p.fe = pf[0];
            r.p.d_e = A;
            r.p.d_a = 1;
            r.p.d_t = n1;
        }
        out.push_back(c);
        out.push_back(r);
        return;
    }
    Pass x, y, z;
    x.p = y.p = z.p = blank();
    // first dimension: rows of the whole grid, kept modes at their start
    x.rows = true;
    x.nt = 1;
    x.p.n = x.p.full = (int)n1;
    x.p.na = (int)(n2 * n3 * nt);
    ends(x, 1, n1, 0, 0, 1, n1, 0, 0, N1, false);
    if (dim == 3) {
        // middle dimension: columns of every plane, in place
        y.rows = false;
        y.nt = 1;
        y.p.n = y.p.full = (int)n2;
        y.p.na = (int)N1;
        y.p.nb = (int)(n3 * nt);
        y.p.col0 = y.p.col1 = 1;
        ends(y, n1, 1, n1 * n2, 0, n1, 1, n1 * n2, 0, N2, false);
    }
    // last dimension: between the grid and the caller's modes
    z.rows = false;
    z.nt = nt;
    z.p.n = z.p.full = (int)(dim == 3 ? n3 : n2);
    z.p.na = (int)N1;
    z.p.nb = (int)(dim == 3 ? N2 : 1);
    z.p.col0 = z.p.col1 = 1;
    if (dim == 3) ends(z, n1 * n2, 1, n1, cells, N1 * N2, 1, N1, modes, N3, true);
    else ends(z, n1, 1, 0, cells, N1, 1, 0, modes, N2, true);
    z.p.scale = 1;
    z.p.fa = pf[0];
    z.p.fb = dim == 3 ? pf[1] : nullptr;
    z.p.fe = dim == 3 ? pf[2] : pf[1];
    if (t1) {
        out.push_back(x);
        if (dim == 3) out.push_back(y);
        out.push_back(z);
    } else {
        out.push_back(z);
        if (dim == 3) out.push_back(y);
        out.push_back(x);
    }
}

// A divisor A of n near its square root with n / A also a line's length.
int four_step(int64_t n)
{
    int best = 0;
    for (int64_t a = 2; a * a <= n; ++a)
        if (n % a == 0) best = (int)a;
    return best;
}

// Passes with the same radix stages share a table of stage factors.
bool same_stages(const FftPass &a, const FftPass &b)
{
    return a.n == b.n && a.radices == b.radices;
}
void add_length(std::vector<FftPass> &lens, const FftPass &p, size_t &vals)
{
    for (const FftPass &l : lens)
        if (same_stages(l, p)) return;
    lens.push_back(p);
    vals += (size_t)p.tw_len;
}

// A pass this small (a line and all values) is bound by the latency of one
// block: the wait for its code and arguments, then stages one after another.
// Four values a thread have a third of the code and four times the waves of
// sixteen: 4.5-5.8 us a pass over 128 x 128 and 256 x 256 grids against
// 5.2-7.4 with 8 values and 5.6-9.7 with 16.  Over 512 x 512 the extra stages
// cost more (5.9-7.4 us against 5.6-6.8 with 8 values).
constexpr long long kSmallPass = 1LL << 17;
constexpr int kSmallLine = 256;

// Radix stages and block shape; fewer values per thread unless the block then
// holds too few lines or the line needs more stages.
bool shape(Pass &q, int prec, bool table, int &V)
{
    const int norm = fft_values(prec);
    FftPass base = q.p;
    if (!fft_line(q.p.n, norm, base)) return false;
    const bool small = q.p.n <= kSmallLine &&
                       (long long)q.p.n * q.p.na * q.p.nb * q.nt <= kSmallPass;
    for (int v : {4, 8, norm, 24}) {
        if (v != norm && (prec != 0 || table)) continue;
        if (v == 4 && !small) continue;
        if (!fft_line(q.p.n, v, q.p) || (v == 8 && q.p.np > base.np && v < norm)) continue;
        if (fft_tile(q.p, prec, q.rows, (long long)q.p.nb * q.nt)) {
            V = v;
            return true;
        }
    }
    return false;
}

}  // namespace

int FftPlan::make(int dim, const int64_t *N, const int *n, int64_t nt, int prec_,
                  const void *const pf[3], const FftAlloc &alloc, hipStream_t s)
{
    prec = prec_;
    ok = false;
    for (auto &d : dir) d.clear();
    const int fourA = dim == 1 && n[0] > kOneLine ? four_step(n[0]) : 0;
    int64_t rows = nt;
    for (int d = 1; d < dim; ++d) rows *= n[d];
    if (rows > 2147483647LL || (dim == 1 && n[0] > kOneLine && !fourA)) return MNUFFT_OK;
    std::vector<Pass> ps[2];
    for (int t = 0; t < 2; ++t) passes_of(t + 1, dim, N, n, nt, pf, 0, 0, fourA, ps[t]);
    for (int t = 0; t < 2; ++t)
        for (Pass &q : ps[t]) {
            FftStep st;
            if (!shape(q, prec, false, st.V)) return MNUFFT_OK;
            st.p = q.p;
            st.form = q.form;
            st.src = q.src;
            st.dst = q.dst;
            st.rotate = q.rotate;
            st.tiles = (long long)q.p.ta * q.p.nb * q.nt;
            if (st.tiles > 2147483647LL) return MNUFFT_OK;
            dir[t].push_back(st);
        }
    // twiddle tables: one per length, and the two-step one of a long line
    const size_t csz = prec == 0 ? 8 : 16;
    std::vector<FftPass> lens;
    size_t vals = 0;
    for (auto &d : dir)
        for (const FftStep &st : d) add_length(lens, st.p, vals);
    const int coarse = fourA ? (int)((n[0] + kTw4 - 1) / kTw4) : 0;
    const size_t total = vals + (fourA ? (size_t)kTw4 + coarse : 0);
    void *tw = nullptr;
    int rc = alloc(&tw, total * csz);
    if (rc) return rc;
    size_t at = 0;
    for (const FftPass &len : lens) {
        void *t = (char *)tw + at * csz;
        if (launch_stage_twiddle(prec, len, t, s) != hipSuccess) return MNUFFT_ERR_HIP;
        for (auto &d : dir)
            for (FftStep &st : d)
                if (same_stages(st.p, len)) st.p.tw = t;
        at += len.tw_len;
    }
    if (fourA) {
        void *t = (char *)tw + at * csz;
        if (launch_twiddle(prec, kTw4, 1, (double)n[0], t, s) != hipSuccess ||
            launch_twiddle(prec, coarse, kTw4, (double)n[0], (char *)t + kTw4 * csz, s) !=
                hipSuccess)
            return MNUFFT_ERR_HIP;
        for (auto &d : dir)
            for (FftStep &st : d)
                if (st.rotate) st.p.tw4 = t;
    }
    work_cells = fourA ? n[0] * nt : 0;
    ok = true;
    return MNUFFT_OK;
}

int FftPlan::run(int type, int sign, void *grid, void *modes, void *work, hipStream_t s) const
{
    void *buf[3] = {grid, modes, work};
    for (const FftStep &st : dir[type - 1]) {
        FftPass p = st.p;
        p.inv = sign > 0;
        if (launch_fft_lines(prec, st.V, st.form, p, nullptr, 0, st.tiles, p.threads, p.lds, buf[st.src],
                             buf[st.dst], s) != hipSuccess)
            return MNUFFT_ERR_HIP;
    }
    return MNUFFT_OK;
}

int FftBatch::make(int type, int dim, int iflag, const std::vector<TGeom> &geo, int prec_,
                   const void *const pf[3], const FftAlloc &alloc, hipStream_t s)
{
    prec = prec_;
    ok = false;
    const size_t csz = prec == 0 ? 8 : 16, rsz = csz / 2;
    std::vector<FftPass> tab[3];
    for (const TGeom &g : geo) {
        const int64_t N[3] = {g.N[0], g.N[1], g.N[2]};
        const void *f[3];
        for (int d = 0; d < 3; ++d) f[d] = (const char *)pf[d] + (size_t)g.p_off[d] * rsz;
        std::vector<Pass> ps;
        passes_of(type, dim, N, g.n, 1, f, g.grid_off, g.mode_off, 0, ps);
        steps = (int)ps.size();
        for (int k = 0; k < steps; ++k) {
            int V = 0;
            if (!shape(ps[k], prec, true, V)) return MNUFFT_OK;
            FftPass p = ps[k].p;
            p.inv = iflag > 0;
            form[k] = ps[k].form;
            src[k] = ps[k].src;
            dst[k] = ps[k].dst;
            if (tiles[k] > 2147483647LL) return MNUFFT_OK;
            p.tile0 = (int)tiles[k];
            tiles[k] += (long long)p.ta * p.nb * ps[k].nt;
            threads[k] = std::max(threads[k], p.threads);
            lds[k] = std::max(lds[k], p.lds);
            tab[k].push_back(p);
        }
    }
    std::vector<FftPass> lens;
    size_t vals = 0;
    for (int k = 0; k < steps; ++k) {
        if (tiles[k] > 2147483647LL) return MNUFFT_OK;
        for (const FftPass &p : tab[k]) add_length(lens, p, vals);
    }
    void *tw = nullptr;
    int rc = alloc(&tw, vals * csz);
    if (rc) return rc;
    size_t at = 0;
    for (const FftPass &len : lens) {
        void *t = (char *)tw + at * csz;
        if (launch_stage_twiddle(prec, len, t, s) != hipSuccess) return MNUFFT_ERR_HIP;
        for (int k = 0; k < steps; ++k)
            for (FftPass &p : tab[k])
                if (same_stages(p, len)) p.tw = t;
        at += len.tw_len;
    }
    for (int k = 0; k < steps; ++k) {
        ntab = (int)tab[k].size();
        void *d = nullptr;
        if ((rc = alloc(&d, tab[k].size() * sizeof(FftPass)))) return rc;
        if (hipMemcpy(d, tab[k].data(), tab[k].size() * sizeof(FftPass), hipMemcpyHostToDevice) !=
            hipSuccess)
            return MNUFFT_ERR_HIP;
        table[k] = (const FftPass *)d;
    }
    if (hipStreamSynchronize(s) != hipSuccess) return MNUFFT_ERR_HIP;
    ok = true;
    return MNUFFT_OK;
}

int FftBatch::run(void *grid, void *modes, hipStream_t s) const
{
    void *buf[2] = {grid, modes};
    for (int k = 0; k < steps; ++k)
        if (launch_fft_lines(prec, fft_values(prec), form[k], FftPass{}, table[k], ntab, tiles[k], threads[k], lds[k],
                             buf[src[k]], buf[dst[k]], s) != hipSuccess)
            return MNUFFT_ERR_HIP;
    return MNUFFT_OK;
}

}  // namespace host
}  // namespace mn
