// Host planning of the hybrid reconstruction: range grid, reference
// wavenumbers, NUFFT parameters, back-projection tiling, workspace layout.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "internal.hpp"

namespace pl {
namespace {

size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

// The n / 2 positive Gauss-Legendre nodes on [-1, 1] and their weights, n
// even (Newton iteration on P_n).
void gauss_legendre(int n, double* x, double* w) {
    for (int i = 0; i < n / 2; ++i) {
        double z = std::cos(kPi * (i + 0.75) / (n + 0.5));
        double dp = 1.0;
        for (int it = 0; it < 100; ++it) {
            double p0 = 1.0, p1 = z;
            for (int k = 2; k <= n; ++k) {
                const double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
                p0 = p1;
                p1 = p2;
            }
            if (n == 1) p0 = 1.0, p1 = z;
            dp = n * (z * p1 - p0) / (z * z - 1.0);
            const double dz = p1 / dp;
            z -= dz;
            if (std::fabs(dz) < 1e-16) break;
        }
        x[i] = z;
        w[i] = 2.0 / ((1.0 - z * z) * dp * dp);
    }
}

// Distance from a point to the axis-aligned rectangle [x0,x1] x [y0,y1].
double dist_to_rect(double px, double py, double x0, double x1, double y0, double y1) {
    const double cx = std::min(std::max(px, x0), x1), cy = std::min(std::max(py, y0), y1);
    return std::hypot(px - cx, py - cy);
}

// Spreading kernel of the NUFFT for the plan's n_l and n_fine; sigma: the
// range grid's oversampling.
int set_spreading(HybridPlan* plan, double sigma) {
    HybridPlan& p = *plan;
    // Exponential-of-semicircle kernel exp(beta (sqrt(1 - z^2) - 1)) of
    // width W (Barnett, Magland, af Klinteberg 2019).  For the 2x fine grid:
    // W = ceil(log10(1/tol)) + 1, beta = 2.30 W.  For an upsampling factor
    // s = n_fine / n_l below 2, their error estimate exp(-pi W sqrt(1 - 1/s))
    // gives W = ceil(ln(1/tol) / (pi sqrt(1 - 1/s))), and beta =
    // 0.97 pi W (1 - 1/(2 s)).
    const double ups = static_cast<double>(p.n_fine) / p.n_l;
    if (ups >= 1.999) {
        p.W = std::max(2, static_cast<int>(std::ceil(std::log10(1.0 / p.tol))) + 1);
        p.W = std::min(p.W, 16);
        p.beta = 2.30 * p.W;
    } else {
        p.W = std::max(2, static_cast<int>(std::ceil(std::log(1.0 / p.tol) / (kPi * std::sqrt(1.0 - 1.0 / ups)))));
        p.W = std::min(p.W, 16);
        p.beta = 0.97 * kPi * p.W * (1.0 - 0.5 / ups);
    }
    p.h = 0.5 * p.W;
    if (p.n_fine / sigma + 2 * p.W + 2 >= p.n_fine) return fail(PL_EUNSUPPORTED, "fine grid too short");
    // quadrature of the kernel's transform: an even integrand, so the positive
    // nodes of an even rule, their weights doubled and times the kernel
    p.n_gl = std::min(2 * kMaxGL, 4 * p.W + 16) / 2;
    gauss_legendre(2 * p.n_gl, p.gl_x, p.gl_w);
    for (int q = 0; q < p.n_gl; ++q)
        p.gl_w[q] *= 2.0 * std::exp(p.beta * (std::sqrt(1.0 - p.gl_x[q] * p.gl_x[q]) - 1.0));
    return PL_OK;
}

// Workspace layout (byte offsets) of the plan: what a call writes first, then
// its tables, from byte tables_from on if that is later.
int set_layout(HybridPlan* plan, size_t tables_from = 0) {
    HybridPlan& p = *plan;
    const size_t nch = p.n_ch, nz = p.n_z, nf = p.n_f, npix = static_cast<size_t>(p.nx) * p.ny;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off = align256(off + bytes);
        return o;
    };
    // the window form's pieces take the place of the spectrum, which no step
    // after the range compression reads
    const size_t part = p.bp_window ? p.part_pieces * kWindowPieceBytes : 0;
    p.off_spec = take(std::max(nch * nz * nf * 8, part));
    p.off_q = take(nch * nz * static_cast<size_t>(p.n_l) * 8);
    p.off_G = take(npix * nz * 8);
    p.off_part = p.bp_window ? p.off_spec : take(backproject_mfma_part_bytes(p));
    p.off_smax = take(p.bp_window ? kSpectrumMaxParts * sizeof(float) : 0);
    off = std::max(off, align256(tables_from));
    // not the last table: the window form reads a carrier's 8 bytes as 16
    p.off_tiles = take(tile_table_bytes(p));
    p.off_llo = take(nch * 8);
    p.off_lref = take(nch * 8);
    p.off_zfft = take(p.zfft.bytes);
    p.off_tw_fine = take(static_cast<size_t>(p.n_fine) * 8);
    p.off_deap = take(static_cast<size_t>(p.n_l) * 4);
    p.off_kp = take(nz * nf * 8);
    p.off_wk = take(nz * nf * 4);
    p.off_krz = take(nz * 8);
    p.n_chp = (p.n_ch + 31) / 32 * 32;
    p.n_fp = (p.n_f + 15) / 16 * 16;
    if (p.precision != PL_PREC_FP32) {
        if (p.n_fp > 128)
            return fail(PL_EUNSUPPORTED, "MFMA range compression supports up to 128 frequencies");
        p.off_mfma_a = take(nz * static_cast<size_t>(p.n_chp) * 4);
        p.off_qexp = take(4 * (kProfileScaleParts + 1));
        p.off_mfma_b = take(nz * static_cast<size_t>(p.n_chp) * 4 * p.n_fp * 2);
    } else {
        p.off_mfma_a = off;
        p.off_mfma_b = off;
        p.off_qexp = off;
    }
    p.total = off;
    return PL_OK;
}

// Weights of the window back-projection: the least-squares interpolator of
// e^{j th x} from the eight samples at s - 3.5, for positions |x| <= xm and
// th spread evenly over each block's band [-X_b, X_b] (X_b = half band x du),
// block b's squared error counted share_b times.  Its normal matrix and
// right-hand side are means of sinc(X_b (s - s')) and sinc(X_b (x - s)); the
// symmetry w_{7-s}(x) = w_s(-x) splits them into 4 x 4 systems for the even
// and odd parts, which are solved at kWindowDegree Chebyshev nodes of x^2 and
// fitted by polynomials in z = 2 x^2 / xm^2 - 1 (w = E + x O; in z their terms
// stay near the size of the weights, while powers of x^2 cancel and would cost
// two digits in float32).
struct WindowWeights {
    double even[kWindowDegree][4], odd[kWindowDegree][4];
};

// sinc(X (x - s)) for s = 0 .. 7, the sine turned by X from each to the next
void sincs(double X, double x, double (&out)[8]) {
    const double cs = std::cos(X), sn = std::sin(X);
    double c = std::cos(X * x), v = std::sin(X * x);
    for (int s = 0; s < 8; ++s) {
        const double y = X * (x - s);
        out[s] = std::fabs(y) < 1e-6 ? 1.0 - y * y / 6.0 : v / y;
        const double t = c * cs + v * sn;
        v = v * cs - c * sn;
        c = t;
    }
}

// The blocks' sinc values that a design takes: the whole sample distances
// from 0, and at its positions.
constexpr int kDesignRows = kWindowDegree + 1;
struct DesignSincs {
    double node[kWindowDegree], x[kWindowDegree];
    std::vector<double> v;   // [block][row][8]
};

DesignSincs design_sincs(const std::vector<double>& X, double xm) {
    DesignSincs d;
    for (int i = 0; i < kWindowDegree; ++i) {
        d.node[i] = std::cos(kPi * (i + 0.5) / kWindowDegree);
        d.x[i] = std::sqrt(0.5 * (1.0 + d.node[i]) * (xm * xm));
    }
    d.v.resize(X.size() * kDesignRows * 8);
    for (size_t b = 0; b < X.size(); ++b)
        for (int i = 0; i < kDesignRows; ++i) {
            double row[8];
            sincs(X[b], i ? d.x[i - 1] + 3.5 : 0.0, row);
            std::copy(row, row + 8, &d.v[(b * kDesignRows + i) * 8]);
        }
    return d;
}

// means of one row over the blocks by the blocks' shares (none: equal ones)
void mean_sincs(const DesignSincs& d, const std::vector<double>& share, int row, double (&out)[8]) {
    double n = 0.0;
    for (double& o : out) o = 0.0;
    for (size_t b = 0; b < d.v.size() / (kDesignRows * 8); ++b) {
        const double f = share.empty() ? 1.0 : share[b];
        for (int s = 0; s < 8; ++s) out[s] += f * d.v[(b * kDesignRows + row) * 8 + s];
        n += f;
    }
    for (double& o : out) o /= n;
}

// b = A^-1 b by elimination with row exchanges
template <int N>
void solve(double (&A)[N][N], double (&b)[N]) {
    for (int i = 0; i < N; ++i) {
        int piv = i;
        for (int r = i + 1; r < N; ++r)
            if (std::fabs(A[r][i]) > std::fabs(A[piv][i])) piv = r;
        for (int c = 0; c < N; ++c) std::swap(A[i][c], A[piv][c]);
        std::swap(b[i], b[piv]);
        for (int r = i + 1; r < N; ++r) {
            const double f = A[r][i] / A[i][i];
            for (int c = i; c < N; ++c) A[r][c] -= f * A[i][c];
            b[r] -= f * b[i];
        }
    }
    for (int i = N - 1; i >= 0; --i) {
        for (int c = i + 1; c < N; ++c) b[i] -= A[i][c] * b[c];
        b[i] /= A[i][i];
    }
}

void window_design(const DesignSincs& d, const std::vector<double>& share, WindowWeights* out) {
    constexpr int D = kWindowDegree;
    double g[8];   // mean sinc at whole sample distances
    mean_sincs(d, share, 0, g);
    double E[D][4], O[D][4];
    for (int i = 0; i < D; ++i) {
        double b[8];
        mean_sincs(d, share, i + 1, b);
        for (int par = 0; par < 2; ++par) {
            const double sg = par ? -1.0 : 1.0;
            double A[4][4], r[4];
            for (int s = 0; s < 4; ++s) {
                for (int t = 0; t < 4; ++t) A[s][t] = g[std::abs(s - t)] + sg * g[7 - s - t];
                A[s][s] += 1e-13;   // below the rounding of the FP16 pairs squared
                r[s] = 0.5 * (b[s] + sg * b[7 - s]);
            }
            solve(A, r);
            for (int s = 0; s < 4; ++s) (par ? O : E)[i][s] = par ? r[s] / d.x[i] : r[s];
        }
    }
    for (int par = 0; par < 2; ++par)
        for (int s = 0; s < 4; ++s) {
            double V[D][D], v[D];
            for (int i = 0; i < D; ++i) {
                double pw = 1.0;
                for (int k = 0; k < D; ++k) V[i][k] = pw, pw *= d.node[i];
                v[i] = (par ? O : E)[i][s];
            }
            solve(V, v);
            for (int k = 0; k < D; ++k) (par ? out->odd : out->even)[k][s] = v[k];
        }
}

// The eight weights at position x.
void window_weights(const WindowWeights& wt, double x, double xm, double (&w)[8]) {
    const double z = 2.0 * x * x / (xm * xm) - 1.0;
    for (int s = 0; s < 4; ++s) {
        double ev = 0.0, od = 0.0;
        for (int k = kWindowDegree - 1; k >= 0; --k) {
            ev = ev * z + wt.even[k][s];
            od = od * z + wt.odd[k][s];
        }
        w[s] = ev + x * od;
        w[7 - s] = ev - x * od;
    }
}

// Squared error of these weights in each block's band, mean over the positions
// |x| <= xm, polynomials included: sums of sinc(X_b (s - s')) and
// sinc(X_b (x - s)) as in the design.
std::vector<double> window_error(const std::vector<double>& X, const DesignSincs& d, double xm,
                                 const WindowWeights& wt) {
    constexpr int NX = 9;
    std::vector<double> e2(X.size(), 0.0);
    for (int i = 0; i < NX; ++i) {
        const double x = xm * (i + 0.5) / NX;
        double w[8], lag[8] = {}, v[8];   // lag[d]: products of weights d samples apart
        window_weights(wt, x, xm, w);
        for (int s = 0; s < 8; ++s)
            for (int t = 0; t < 8; ++t) lag[std::abs(s - t)] += w[s] * w[t];
        for (size_t b = 0; b < X.size(); ++b) {
            const double* g = &d.v[b * kDesignRows * 8];
            sincs(X[b], x + 3.5, v);
            double e = 1.0;
            for (int s = 0; s < 8; ++s) e += lag[s] * g[s] - 2.0 * w[s] * v[s];
            e2[b] += std::max(e, 0.0) / NX;
        }
    }
    return e2;
}

// rms of the first n squared errors
double rms(const std::vector<double>& e2, size_t n) {
    double s = 0.0;
    for (size_t b = 0; b < n; ++b) s += e2[b];
    return std::sqrt(s / static_cast<double>(n));
}

// The phase steps per sample th and, at each, the turn e^{j th} and the turns
// at the positions x = xm (j + 1/2) / kCells from the window's first sample.
constexpr int kCells = 9, kPhase = 32;
struct PhaseTurns {
    double cs[kPhase], sn[kPhase], c[kPhase][kCells], s[kPhase][kCells];
};

void phase_turns(double most, double xm, PhaseTurns* t) {
    for (int i = 0; i < kPhase; ++i) {
        const double th = (i + 0.5) / kPhase * most;
        t->cs[i] = std::cos(th);
        t->sn[i] = std::sin(th);
        for (int j = 0; j < kCells; ++j) {
            const double ph = th * (xm * (j + 0.5) / kCells + 3.5);
            t->c[i][j] = std::cos(ph);
            t->s[i][j] = std::sin(ph);
        }
    }
}

// The weights' squared error at each phase step, mean over the positions by
// the shares at[j].
void window_error(const PhaseTurns& p, double xm, const double (&at)[kCells], const WindowWeights& wt, double* e2) {
    double w[kCells][8];
    for (int j = 0; j < kCells; ++j) window_weights(wt, xm * (j + 0.5) / kCells, xm, w[j]);
    for (int i = 0; i < kPhase; ++i) {
        const double cs = p.cs[i], sn = p.sn[i];
        e2[i] = 0.0;
        for (int j = 0; j < kCells; ++j) {
            if (at[j] == 0.0) continue;
            // sum_s w_s e^{j th (s - 3.5 - x)} - 1 by the powers of e^{j th}
            double re = 0.0, im = 0.0;
            for (int s = 7; s >= 0; --s) {
                const double t = re * cs - im * sn + w[j][s];
                im = re * sn + im * cs;
                re = t;
            }
            const double c0 = p.c[i][j], s0 = p.s[i][j];
            const double dr = re * c0 + im * s0 - 1.0, di = im * c0 - re * s0;
            e2[i] += at[j] * (dr * dr + di * di);
        }
    }
}

// How often a pixel's position in its group's window falls into each of the
// cells: nine groups over the image and eight channels over the array.
void window_positions(const pl_geometry* g, const HybridPlan& p, double xm, double (&at)[kCells]) {
    for (double& a : at) a = 0.0;
    const double centre = 0.5 * p.win_span - 3.5;
    for (int i = 0; i < 8; ++i) {
        const int c = (2 * i + 1) * p.n_ch / 16;
        const double *t = &g->tx[2 * c], *r = &g->rx[2 * c];
        for (int k = 0; k < 9; ++k) {
            const int gx = (p.nx + 3) / 4 * (2 * (k % 3) + 1) / 6, gy = (p.ny + 3) / 4 * (2 * (k / 3) + 1) / 6;
            double v[16], low = 1e300;
            for (int q = 0; q < 16; ++q) {
                const double x = p.x0 + (4 * gx + q % 4) * p.dx, y = p.y0 + (4 * gy + q / 4) * p.dy;
                const double lt = std::sqrt((x - t[0]) * (x - t[0]) + (y - t[1]) * (y - t[1]));
                const double lr = p.mode == PL_MONO ? lt : std::sqrt((x - r[0]) * (x - r[0]) + (y - r[1]) * (y - r[1]));
                v[q] = (lt + lr) / p.du;
                low = std::min(low, v[q]);
            }
            const double start = std::rint((low + centre) / p.win_step) * p.win_step;
            for (double u : v) at[std::min(kCells - 1, static_cast<int>(std::fabs(u - start - 3.5) / xm * kCells))] += 1.0 / 1152;
        }
    }
}

// The window plan of a whole FP32 call (see k_backproject_window.hip), or
// false where it does not apply: other precisions, methods or references, an
// option that asks for a kernel or its shape, an interpolation or an
// oversampling of the caller's own, or a pixel pitch too coarse for eight
// samples per 4x4 group.
//
// The range step: a group's ranges span at most gspan = 2 |(3 dx, 3 dy)|
// (|grad l| <= 2); the step is the widest of five (gspan = 3.4 .. 5.66
// samples) at which equal shares of all blocks give an estimated interpolation
// error of 0.55 of the B-spline's at the caller's oversampling over the same
// bands (even window starts) or 0.9 of it (any start), and at most 1.5 of it
// over the lower half of |k_z|.
//
// The shares: the B-spline's error falls as the fourth power of a block's
// band, these weights' hardly, and an echo's energy lies at the |k_z| its
// aperture sees, from 0 up: with equal shares the image was less exact than
// the B-spline path's where the lowest blocks are much narrower than the rest
// (16 of 368 problems of 69 .. 512 scan positions and 2.2 .. 5.6 mm pixels, by
// up to 2.4, 11 of them with a 3 mm scan step; an echo at k_z = 0 alone in 82,
// by up to 3.7).  Shares h_b^(-8 gamma) (h_b the block's half band) trade error
// of the wide bands for the narrow ones'.  For each gamma both forms' squared
// errors are summed over the k' of every propagating (frequency, bin), in the
// blocks each form has and at the positions in the window that occur, from
// k_z = 0 up to six fractions of |k_z|; the first gamma at which the largest of
// the six ratios is at most 0.7 is taken, or the one where it is smallest,
// which has to be at most 1.05 (4 of the 368, at 1.3 to 2.4 before, keep the
// other plan).  The 364 have 0.36 of the B-spline path's error in the mean,
// five of them more than it (1.14 .. 1.49 of errors of 1.2 .. 2.6e-6), and at
// k_z = 0 alone 39 (up to 1.75).  With all positions alike in the estimate 10
// of 260 were refused, most of them below 1.
//
// base: the call's plan in FP32; held: the plan that runs otherwise.  own_workspace:
// one that only such calls use; else the tables lie past all that
// other calls with the same arguments (the adjoint, the steps) write.
bool window_plan(const pl_geometry* g, const pl_image_grid* grid, const HybridPlan& base, const HybridPlan& held,
                 bool own_workspace, HybridPlan* out) {
    if (base.precision != PL_PREC_FP32 || base.range_method != PL_RANGE_NUFFT || base.ref_mode != PL_REF_BAND_CENTRE ||
        base.interp != PL_INTERP_BSPLINE4 || base.sigma_l > 6.0 || base.force_tile || base.force_tile_y ||
        base.force_kpl || base.force_waves || base.force_kb || base.force_bp_mfma)
        return false;
    HybridPlan p = base;
    p.bp_window = true;
    p.bp_gather = false;
    p.block = kWindowBins;
    const int n_lo = (p.n_z + 1) / 2;
    p.n_blocks = (n_lo + kWindowBins - 1) / kWindowBins;
    std::vector<double> half(p.n_blocks, 0.0);
    p.half_band = 0.0;
    // k_rho over the propagating frequencies of bins [m0, m1]; empty: hi < lo
    auto band = [&](int m0, int m1, double* lo, double* hi) {
        *lo = 1e300;
        *hi = -1e300;
        for (int m = m0; m <= m1; ++m) {
            const double kz = 2.0 * kPi * m / (p.n_z * g->scan_step), q = 0.25 * kz * kz;
            if (g->k[p.n_f - 1] * g->k[p.n_f - 1] <= q) continue;
            // the first propagating frequency (k rises with f)
            const double kf = *std::partition_point(g->k.begin(), g->k.end(), [&](double k) { return k * k <= q; });
            *lo = std::min(*lo, std::sqrt(kf * kf - q));
            *hi = std::max(*hi, std::sqrt(g->k[p.n_f - 1] * g->k[p.n_f - 1] - q));
        }
    };
    for (int b = 0; b < p.n_blocks; ++b) {
        // |k_z| of bins m and mirrors n - 1 - m (which is -(m + 1) steps)
        const int m0 = b * kWindowBins, m1 = std::min(n_lo, m0 + kWindowBins) - 1;
        double lo, hi;
        band(m0, m1 < p.n_z / 2 ? m1 + 1 : m1, &lo, &hi);
        p.kref[b] = hi < lo ? 0.0 : 0.5 * (lo + hi);
        half[b] = hi < lo ? 0.0 : 0.5 * (hi - lo);
        p.half_band = std::max(p.half_band, half[b]);
    }
    if (!(p.half_band > 0)) return false;   // one frequency, no k_z spread
    // Small images of which the 16x16 tiles and 32-bin blocks would be more
    // than a third padding stay with the vector kernels.  The line was drawn by
    // seven of 220 problems that the window form slowed by 1 to 12 %, and is on
    // the safe side: of 691 timed problems that it keeps back 86 would lose
    // more than 2 %, and 539 would gain more than 5 % (median 1.2 times, at
    // most 3.7).  Of 509 that pass, 54 lose (2 to 29 %, half of them calls
    // below 100 us) and have up to 6 times smaller errors.
    const double pixels = static_cast<double>(p.nx) * p.ny, tiles = std::ceil(p.nx / 16.0) * std::ceil(p.ny / 16.0);
    if (pixels * n_lo < 0.66 * tiles * 256 * kWindowBins * p.n_blocks && pixels * p.n_z * p.n_ch < 3.2e8) return false;
    if (p.half_band * std::hypot(3.0 * grid->dx, 3.0 * grid->dy) * 2.0 / 5.66 > 1.1) return false;   // far over the bound
    // the B-spline's error, sqrt(2) (k' du / 2 pi)^4 at k': over all bands,
    // and over the lower half of |k_z|, where a scene's echo is strongest
    auto spline_error = [](const std::vector<double>& h, size_t n, double du) {
        double e2 = 0.0;
        for (size_t b = 0; b < n; ++b) e2 += 2.0 * std::pow(h[b] * du / (2.0 * kPi), 8) / 9.0;
        return std::sqrt(e2 / n);
    };
    const int n_low = (p.n_blocks + 1) / 2;
    const double base_err = spline_error(half, half.size(), base.du), base_low = spline_error(half, n_low, base.du);
    // Where the B-spline itself is off by about its largest estimate (2.3e-5,
    // a block as wide as the band of k', scans of up to some 70 positions) the
    // two forms' images would differ by more than 2e-5: the other plan stays.
    // The matrix-core modes' own blocks are wider.
    std::vector<double> own(half);
    if (held.block != kWindowBins) {
        own.clear();
        for (int m0 = 0; m0 < n_lo; m0 += held.block) {
            double lo, hi;
            band(m0, std::min(m0 + held.block, p.n_z / 2), &lo, &hi);
            own.push_back(hi < lo ? 0.0 : 0.5 * (hi - lo));
        }
    }
    if (spline_error(own, (own.size() + 1) / 2, held.du) > 1.6e-5 || spline_error(own, own.size(), held.du) > 1.9e-5)
        return false;

    const double gspan = std::hypot(3.0 * grid->dx, 3.0 * grid->dy) * 2.0;
    const double spans[5] = {3.4, 3.77, 4.25, 4.85, 5.66};
    WindowWeights w;
    auto admitted = [&](int step, int i) {
        p.win_step = step;
        p.win_span = spans[i];
        p.du = gspan / spans[i];
        p.sigma_used = kPi / (p.half_band * p.du);
        if (p.sigma_used < 1.3) return false;
        std::vector<double> X;
        for (double h : half) X.push_back(h * p.du);
        // positions: half the span, half a step of the window's start, and
        // 1/64 sample and float rounding of the group's lowest position
        const double xm = 0.5 * (spans[i] + step) + 0.02;
        p.win_z = 2.0 / (xm * xm);
        const DesignSincs values = design_sincs(X, xm);
        window_design(values, {}, &w);
        const std::vector<double> e2 = window_error(X, values, xm, w);
        return rms(e2, e2.size()) <= (step == 2 ? 0.55 : 0.9) * base_err && rms(e2, n_low) <= 1.5 * base_low;
    };
    bool found = false;
    for (int step = 2; step >= 1 && !found; --step) {
        if (!admitted(step, 4)) continue;   // the narrowest step
        int lo = 0, hi = 4, last = 4;       // the error falls with the step: the first of the five admitted
        while (lo < hi) {
            const int mid = (lo + hi) / 2;
            last = mid;
            if (admitted(step, mid)) hi = mid;
            else lo = mid + 1;
        }
        found = last == hi || admitted(step, hi);
    }
    if (!found) return false;

    // the shares (see above)
    constexpr double kBelow = 0.7, kMost = 1.05;
    const double fraction[6] = {0.125, 0.25, 0.375, 0.5, 0.75, 1.0};
    double count[6][kPhase] = {}, spline[6] = {}, e2[kPhase];   // kPhase cells of |k'|
    const int last = p.n_z / 2;   // bins m = 0 .. last and -m
    const int fs = std::max(1, p.n_f / 8), ms = std::max(1, last / 64);   // some 8 frequencies, 64 to 128 bins
    for (int m = 0; m <= last; m += ms) {
        const double kz = 2.0 * kPi * m / (p.n_z * g->scan_step), q = 0.25 * kz * kz;
        int part = 0;
        while (part < 5 && m > fraction[part] * last) ++part;
        for (int f = 0; f < p.n_f; f += fs) {
            if (g->k[f] * g->k[f] <= q) continue;
            const double kr = std::sqrt(g->k[f] * g->k[f] - q);
            for (int sg = 0; sg < 2; ++sg) {
                const int kap = sg && m ? p.n_z - m : m;
                const double kw = std::fabs(kr - p.kref[std::min(kap, p.n_z - 1 - kap) / kWindowBins]);
                const double x = (kr - base.kref[kap / base.block]) * base.du / (2.0 * kPi);
                ++count[part][std::min(kPhase - 1, static_cast<int>(kw / p.half_band * kPhase))];
                spline[part] += 2.0 * (x * x * x * x) * (x * x * x * x);
            }
        }
    }
    std::vector<double> X;
    for (double h : half) X.push_back(h * p.du);
    const double xm = 0.5 * (p.win_span + p.win_step) + 0.02;
    double at[kCells], least = 1e300;
    window_positions(g, p, xm, at);
    const DesignSincs values = design_sincs(X, xm);
    PhaseTurns turns;
    phase_turns(p.half_band * p.du, xm, &turns);
    for (double gamma : {0.0, 0.5, 0.75, 1.0, 1.25, 1.5, 1.75, 2.0, 2.5}) {
        std::vector<double> share;
        for (double h : half) share.push_back(std::pow(std::max(h / p.half_band, 0.25), -8.0 * gamma));
        WindowWeights t = w;   // equal shares: as the step was chosen
        if (gamma > 0) window_design(values, share, &t);
        window_error(turns, xm, at, t, e2);
        double worst = 0.0, sw = 0.0, ss = 0.0;
        for (int i = 0; i < 6; ++i) {
            for (int j = 0; j < kPhase; ++j) sw += count[i][j] * e2[j];
            ss += spline[i];
            const double r = std::sqrt(sw / ss);
            if (!(r <= worst)) worst = r;   // also one that is not a number
        }
        if (worst < least) {
            least = worst;
            w = t;
        }
        if (least <= kBelow) break;
    }
    if (!(least <= kMost)) return false;
    for (int k = 0; k < kWindowDegree; ++k)
        for (int s = 0; s < 4; ++s) {
            p.win_even[k][s] = static_cast<float>(w.even[k][s]);
            p.win_odd[k][s] = static_cast<float>(w.odd[k][s]);
        }

    // staged rows: every group's window of a 16x16 tile, from a start on a
    // multiple of four samples (the tile table's window start)
    p.tile_x = p.tile_y = 16;
    p.tiles_x = (p.nx + 15) / 16;
    p.tiles_y = (p.ny + 15) / 16;
    p.waves = 8;
    const double reach = 2.0 * std::hypot(15.0 * grid->dx, 15.0 * grid->dy) / p.du;
    const int lead = p.win_step == 2 ? 2 : 0;   // half the rows are staged from two samples earlier
    const int chunks = std::max(8, (static_cast<int>(std::ceil(reach - p.win_span + 9.2 + p.win_step)) + 3 + lead + 3) / 4);
    if (chunks > 9) return false;
    p.window = 4 * chunks;
    p.window_pad = 2 * chunks + 1;
    // eight samples beyond the image's ranges on both sides (the windows of
    // groups that reach past the image's edge), and four before the first
    // staged row
    p.lo_margin = 12;
    p.n_l = std::max(static_cast<int>(std::ceil(p.span / p.du)) + 21, p.window + 4);
    p.n_l = (p.n_l + 3) & ~3;
    const int want = static_cast<int>(std::ceil(kNufftUpsample * p.n_l));
    p.n_fine = 0;
    for (int r = std::max(2, (want + 63) / 64); r <= 32 && !p.n_fine; ++r)
        if (is_fft_friendly(r)) p.n_fine = 64 * r;
    if (!p.n_fine || static_cast<unsigned long long>(p.n_z) * p.n_l * 8 >= (1ull << 31)) return false;
    factor_radices(p.n_fine, &p.fine_rad);
    if (set_spreading(&p, p.sigma_used)) return false;
    // |q| <= n_f k_max sqrt(2) (largest |S| part), a tenth for the NUFFT's error
    p.log2_gain = static_cast<int>(std::ceil(std::log2(1.6 * p.n_f * g->k[p.n_f - 1])));

    // split items' partial spectra: those of the launch's tail split on the
    // card's kWindowSlots resident workgroups, none where it splits nothing,
    // and no more than the static scratch has room for (in the spectrum's
    // place) where it holds the problem
    p.part_pieces = 0;
    if (set_layout(&p)) return false;
    const long long items = static_cast<long long>(p.tiles_x) * p.tiles_y * p.n_blocks, tail = items % kWindowSlots;
    long long pieces = 0;   // per split item
    if (tail > 0 && 2 * tail <= kWindowSlots) pieces = std::min<long long>(kWindowSlots / tail, (p.n_ch + 1) / 2);
    const size_t scratch = static_cast<size_t>(PL_STATIC_SCRATCH_BYTES);
    if (held.total <= scratch) {
        if (p.total > scratch) return false;
        const size_t room = scratch - p.total + static_cast<size_t>(p.n_ch) * p.n_z * p.n_f * 8;
        if (pieces) pieces = std::min<long long>(pieces, room / kWindowPieceBytes / tail);
    }
    p.part_pieces = pieces >= 2 ? static_cast<int>(tail * pieces) : 0;
    if (set_layout(&p, own_workspace ? 0 : held.total)) return false;
    *out = p;
    return true;
}

}  // namespace

int make_plan(const pl_geometry* g, const pl_image_grid* grid, const pl_hybrid_opts* opts,
              HybridPlan* out) {
    if (!g || !grid || !out) return fail(PL_EINVAL, "null geometry, grid or plan");
    if (grid->nx < 1 || grid->ny < 1 || !(grid->dx > 0) || !(grid->dy > 0) ||
        !std::isfinite(grid->x0) || !std::isfinite(grid->y0))
        return fail(PL_EINVAL, "image grid needs nx, ny >= 1 and dx, dy > 0");
    if (static_cast<long long>(grid->nx) * grid->ny > (1LL << 26))
        return fail(PL_EUNSUPPORTED, "image grid has more than 2^26 pixels");
    HybridPlan p;
    p.mode = g->mode;
    p.n_ch = g->n_ch;
    p.n_z = g->n_scan;
    p.n_f = g->n_freq;
    p.scan_step = g->scan_step;
    p.nx = grid->nx;
    p.ny = grid->ny;
    p.x0 = grid->x0;
    p.y0 = grid->y0;
    p.dx = grid->dx;
    p.dy = grid->dy;
    if (opts) {
        p.precision = opts->precision;
        p.interp = opts->interp;
        if (opts->l_oversample != 0) p.sigma_l = opts->l_oversample;
        if (opts->nufft_tol != 0) p.tol = opts->nufft_tol;
        p.force_tile = opts->tile;
        p.force_kpl = opts->kz_per_lane;
        p.force_waves = opts->waves;
        p.force_bp_mfma = opts->mfma_backprojection;
        p.force_tile_y = opts->tile_y;
        p.force_kb = opts->kz_block;
        p.range_method = opts->range_method;
        p.ref_mode = opts->ref_mode;
    }
    if (p.ref_mode != PL_REF_BAND_CENTRE && p.ref_mode != PL_REF_MIN_K)
        return fail(PL_EINVAL, "unknown ref_mode %d", p.ref_mode);
    if (p.ref_mode == PL_REF_MIN_K) {
        // the paper's reference differs per k_z bin: its carrier is formed per
        // term, which only the k_z-per-lane back-projection does
        if (p.range_method != PL_RANGE_NUFFT)
            return fail(PL_EUNSUPPORTED, "ref_mode PL_REF_MIN_K takes the NUFFT range compression");
        if (p.force_bp_mfma > 0)
            return fail(PL_EUNSUPPORTED, "ref_mode PL_REF_MIN_K takes the VALU back-projection");
        if (p.force_kpl > 1 || p.force_kb != 0 || (p.force_waves != 0 && p.force_waves != 4))
            return fail(PL_EUNSUPPORTED, "ref_mode PL_REF_MIN_K runs one k_z bin per lane, 4 wavefronts");
    }
    if (p.force_kpl != 0 && p.force_kpl != 1 && p.force_kpl != 2 && p.force_kpl != 4)
        return fail(PL_EINVAL, "kz_per_lane must be 0, 1, 2 or 4");
    if (p.force_waves != 0 && p.force_waves != 4 && p.force_waves != 8)
        return fail(PL_EINVAL, "waves must be 0, 4 or 8");
    if (p.force_tile != 0 && p.force_tile != 16 && p.force_tile != 8 && p.force_tile != 4 && p.force_tile != 2)
        return fail(PL_EINVAL, "tile must be 0, 16, 8, 4 or 2");
    if (p.force_tile_y != 0 && p.force_tile_y != 16 && p.force_tile_y != 8)
        return fail(PL_EINVAL, "tile_y must be 0, 16 or 8");
    if (p.force_kb != 0 && p.force_kb != 32 && p.force_kb != 64 && p.force_kb != 128)
        return fail(PL_EINVAL, "kz_block must be 0, 32, 64 or 128");
    if (p.precision < PL_PREC_FP32 || p.precision > PL_PREC_FP16)
        return fail(PL_EINVAL, "unknown precision %d", p.precision);
    if (p.range_method != PL_RANGE_NUFFT && p.range_method != PL_RANGE_RESAMPLE)
        return fail(PL_EINVAL, "unknown range_method %d", p.range_method);
    if (p.range_method == PL_RANGE_RESAMPLE) {
        if (p.precision != PL_PREC_FP32)
            return fail(PL_EUNSUPPORTED, "the resampling range compression runs in FP32 only");
        if (p.n_f < 2) return fail(PL_EUNSUPPORTED, "the resampling range compression needs two frequencies");
    }
    if (p.interp < PL_INTERP_BSPLINE4 || p.interp > PL_INTERP_LINEAR)
        return fail(PL_EINVAL, "unknown interpolation %d", p.interp);
    if (!(p.sigma_l >= 2.0 && p.sigma_l <= 64.0)) return fail(PL_EINVAL, "l_oversample must be in [2, 64]");
    if (!(p.tol >= 1e-12 && p.tol <= 1e-2)) return fail(PL_EINVAL, "nufft_tol must be in [1e-12, 1e-2]");
    if (int rc = plan_axis_fft(p.n_z, &p.zfft)) return rc;

    // Dispersion k_rho = sqrt(k^2 - k_z^2 / 4) for the range l = rho_T + rho_R
    // (eq. 18; the monostatic eq. 5 is the same relation with l = 2 rho).
    // One reference wavenumber per block of k_z bins: the centre of the band
    // of k_rho it spans.  The reference cancels exactly between eqs. (8a) and
    // (8b); only the bandwidth of the range profiles depends on it.
    // Reference wavenumber of every k_z block and the range-grid step for a
    // given block size.
    auto set_blocks = [&](int block, double sigma) {
        p.block = std::max(block, kMinBlock);
        p.n_blocks = (p.n_z + p.block - 1) / p.block;  // <= kMaxScan / kMinBlock = kMaxBlocks
        double half_band = 0.0;
        for (int b = 0; b < p.n_blocks; ++b) {
            double lo = 1e300, hi = -1e300;
            for (int kap = b * p.block; kap < std::min(p.n_z, (b + 1) * p.block); ++kap) {
                const int sk = kap < (p.n_z + 1) / 2 ? kap : kap - p.n_z;
                const double kz = 2.0 * kPi * sk / (p.n_z * g->scan_step);
                // k_rho rises with f: its extremes are those of the first
                // propagating frequency and the last
                auto arg = [&](double k) { return k * k - 0.25 * kz * kz; };
                if (arg(g->k[p.n_f - 1]) <= 0) continue;
                const double kf = *std::partition_point(g->k.begin(), g->k.end(), [&](double k) { return arg(k) <= 0; });
                lo = std::min(lo, std::sqrt(arg(kf)));
                hi = std::max(hi, std::sqrt(arg(g->k[p.n_f - 1])));
            }
            if (hi < lo) {
                p.kref[b] = 0.0;
            } else {
                p.kref[b] = 0.5 * (lo + hi);
                half_band = std::max(half_band, 0.5 * (hi - lo));
            }
        }
        if (p.ref_mode == PL_REF_MIN_K) {
            // the paper's k_rho0 = k_rho at the lowest wavenumber k_0 (the
            // smallest real k_rho of the bin where k_0 is evanescent): k' runs
            // over [0, max k_rho - k_rho0], so the range grid resolves the
            // widest such band
            half_band = 0.0;
            for (int kap = 0; kap < p.n_z; ++kap) {
                const int sk = kap < (p.n_z + 1) / 2 ? kap : kap - p.n_z;
                const double kz = 2.0 * kPi * sk / (p.n_z * g->scan_step);
                double lo = -1.0, hi = -1.0;
                for (int f = 0; f < p.n_f; ++f) {
                    const double arg = g->k[f] * g->k[f] - 0.25 * kz * kz;
                    if (arg <= 0) continue;
                    const double kr = std::sqrt(arg);
                    if (lo < 0) lo = kr;
                    hi = kr;
                }
                if (lo >= 0) half_band = std::max(half_band, hi - lo);
            }
        }
        if (half_band <= 0) half_band = 1.0;  // single frequency, no k_z spread
        p.half_band = half_band;
        p.sigma_used = sigma;
        p.du = kPi / (sigma * half_band);
    };

    // MFMA back-projection (BF16 / FP16 modes): tiles of 4x4 pixel groups,
    // each group's taps inside one 16-sample window that starts on a multiple
    // of 4 samples.  |l(p) - l(q)| <= 2 |p - q|, so a group's first tap is at
    // most 3 samples past its window start and its last at most
    // ceil(2 * diagonal / du) + 3 past its first.  The kernel forms each
    // pixel's position in float32 from its tile centre's (error far below
    // 1e-3 samples), so the plan keeps 2 * diagonal / du <= 8.99: a floor
    // taken in float32 then never spreads a group's first taps over more
    // than 9 samples.
    p.bp_mfma = false;
    p.bp_mfma_sp = false;
    if (p.force_bp_mfma > 2) return fail(PL_EINVAL, "mfma_backprojection must be -1, 0, 1 or 2");
    if (p.force_bp_mfma > 0) {
        if (p.precision == PL_PREC_FP32)
            return fail(PL_EUNSUPPORTED, "the MFMA back-projection runs in the BF16 / FP16 modes only");
        // single pass: one FP16 product per pair (scaled FP16 profiles)
        const bool sp = p.force_bp_mfma == 2;
        if (sp && p.precision != PL_PREC_FP16)
            return fail(PL_EUNSUPPORTED, "the single-pass MFMA back-projection runs in the FP16 mode only");
        if (p.force_kpl != 0)
            return fail(PL_EINVAL, "kz_per_lane applies to the VALU back-projection");
        const int tx = p.force_tile ? p.force_tile : 16;
        const int ty = p.force_tile_y ? p.force_tile_y : tx;
        if (!((tx == 8 && ty == 8) || (tx == 16 && (ty == 8 || ty == 16))))
            return fail(PL_EINVAL, "MFMA back-projection tiles are 8x8, 16x8 or 16x16");
        const int kb = p.force_kb ? p.force_kb : 64;
        if (kb == 32) return fail(PL_EINVAL, "the MFMA back-projection takes 64 or 128 k_z bins per workgroup");
        // eight wavefronts (two 4x4 groups each) on the 16x16 and 16x8 tiles
        // with 64 k_z bins: measured fastest on gfx950
        const double gdiag = std::hypot(3.0 * grid->dx, 3.0 * grid->dy);
        set_blocks(kb, p.sigma_l);
        if (2.0 * gdiag / p.du > 8.99) {
            // widest grid step that fits, as long as the oversampling stays >= 4
            const double du_fit = 2.0 * gdiag / 8.99;
            const double sigma_fit = kPi / (du_fit * p.half_band);
            if (sigma_fit >= 4.0) set_blocks(kb, std::min(p.sigma_l, sigma_fit));
        }
        // staged window: every tap of the tile plus alignment (8-sample
        // chunks), and one sample against float rounding
        const double rt = 0.5 * std::hypot((tx - 1) * grid->dx, (ty - 1) * grid->dy);
        const int need = static_cast<int>(std::ceil(4.0 * rt / p.du)) + 7;
        const int nck = std::max(2, (need + 7) / 8);
        const size_t lds = backproject_mfma_lds_bytes(kb, sp);
        if (2.0 * gdiag / p.du <= 8.995 && nck <= 8 && lds <= kMaxLds && p.n_f <= 128) {
            p.bp_mfma = true;
            p.bp_mfma_sp = sp;
            p.tile_x = tx;
            p.tile_y = ty;
            p.window = 8 * nck;  // samples staged per plane and row
            p.window_pad = sp ? 17 : 33;  // LDS row length in 16-byte chunks (2 or 4 planes x 8 + 1)
            p.waves = p.force_waves ? p.force_waves : ((tx * ty >= 128 && kb == 64) ? 8 : 4);
            if (tx * ty == 64 && p.waves == 8)
                return fail(PL_EUNSUPPORTED, "8 wavefronts need a 16x8 or 16x16 MFMA tile");
            if (tx * ty == 256 && kb == 128 && p.waves == 8)
                return fail(PL_EUNSUPPORTED, "8 wavefronts with a 16x16 tile take 64 k_z bins");
        }
    }
    if (p.force_bp_mfma > 0 && !p.bp_mfma)
        return fail(PL_EUNSUPPORTED, "the MFMA back-projection does not fit this grid");
    // VALU back-projection: the pixel-per-lane kernel when its 8x8 tile's
    // window fits (32 k_z bins per workgroup by default: the narrower k'
    // band of a smaller block coarsens the range grid, and with 64 bins the
    // row buffers halve the workgroups per CU), else one k_z bin per lane
    // (one bin per lane by default:
    // more bins per lane make the staged window too large for several
    // resident workgroups per CU).
    p.bp_gather = false;
    if (!p.bp_mfma) {
        if (p.force_tile == 16 || p.force_tile_y != 0)
            return fail(PL_EINVAL, "tile 16 and tile_y apply to the MFMA back-projection");
        if (p.force_kb && (p.force_kb > 64 || p.force_kpl))
            return fail(PL_EINVAL, "the VALU back-projection takes kz_block 32 or 64 (pixel-per-lane kernel)");
        if (p.force_kpl == 0 && (p.force_tile == 0 || p.force_tile == 8) &&
            (p.force_waves == 0 || p.force_waves == 4) && p.ref_mode == PL_REF_BAND_CENTRE) {
            // staged rows start on an even sample (16-byte copies) and hold
            // the window: the taps of every pixel of the 8x8 tile and the
            // sample after them (a pixel reads three aligned chunks around
            // its four taps), ceil(2 reach / du) + 7 samples with reach = 2 rt,
            // and one more against float rounding
            set_blocks(p.force_kb ? p.force_kb : 32, p.sigma_l);
            const double rt = 0.5 * std::hypot(7.0 * grid->dx, 7.0 * grid->dy);
            const int nchk = (static_cast<int>(std::ceil(4.0 * rt / p.du)) + 8 + 1) / 2;  // 2-sample chunks
            const int rows[6] = {12, 14, 18, 24, 32, 40};   // compiled row classes
            int rsc = 0;
            for (int r : rows)
                if (!rsc && nchk <= r) rsc = r;
            if (rsc && backproject_gather_lds_bytes(p.block, rsc) <= kMaxLds) {
                p.bp_gather = true;
                p.tile_x = p.tile_y = 8;
                p.window = 2 * nchk;   // samples staged per row
                p.window_pad = rsc;    // LDS row length in 16-byte chunks
                p.waves = 4;
            }
        }
        if (!p.bp_gather) {
            if (p.force_kb) return fail(PL_EUNSUPPORTED, "kz_block needs the pixel-per-lane back-projection");
            set_blocks(kLanes * (p.force_kpl ? p.force_kpl : 1), p.sigma_l);
        }
    }

    // Range window of every channel over the pixel-centre rectangle.
    const double gx1 = grid->x0 + (grid->nx - 1) * grid->dx, gy1 = grid->y0 + (grid->ny - 1) * grid->dy;
    double span = 0.0;
    for (int c = 0; c < p.n_ch; ++c) {
        const double tx = g->tx[2 * c], ty = g->tx[2 * c + 1], rx = g->rx[2 * c], ry = g->rx[2 * c + 1];
        const double lmin = dist_to_rect(tx, ty, grid->x0, gx1, grid->y0, gy1) +
                            dist_to_rect(rx, ry, grid->x0, gx1, grid->y0, gy1);
        double lmax = 0.0;
        for (int i = 0; i < 4; ++i) {
            const double x = (i & 1) ? gx1 : grid->x0, y = (i & 2) ? gy1 : grid->y0;
            lmax = std::max(lmax, std::hypot(x - tx, y - ty) + std::hypot(x - rx, y - ry));
        }
        span = std::max(span, lmax - lmin);
    }

    p.span = span;

    // k_z-per-lane kernel tile: the staged range window must hold every tap
    // of the tile's pixels (|l(p) - l(centre)| <= 2 * half-diagonal).  Prefer
    // the largest tile whose window fits 64 samples (one staging load per
    // lane and row; the 2x2 fallback allows 128) and whose LDS (window starts
    // + two staged windows of 64 x kz_per_lane rows) fits the workgroup's
    // 160 KiB.
    if (!p.bp_mfma && !p.bp_gather) {
        const int tiles[3][2] = {{8, 8}, {4, 4}, {2, 2}};
        p.window = 0;
        for (int t = 0; t < 3; ++t) {
            if (p.force_tile && tiles[t][0] != p.force_tile) continue;
            const double rt = 0.5 * std::hypot((tiles[t][0] - 1) * grid->dx, (tiles[t][1] - 1) * grid->dy);
            const int wl = static_cast<int>(std::ceil(4.0 * rt / p.du)) + 6;
            const size_t lds = backproject_lds_bytes(p.n_ch, p.block, wl | 1);
            if ((wl <= (t == 2 ? 128 : 64) && lds <= kMaxLds) || t == 2 || p.force_tile) {
                p.tile_x = tiles[t][0];
                p.tile_y = tiles[t][1];
                p.window = wl;
                break;
            }
        }
        p.waves = p.force_waves ? p.force_waves : 4;
        if (p.waves == 8 && p.tile_x != 8)
            return fail(PL_EUNSUPPORTED, "8 wavefronts per workgroup need the 8x8 tile");
        if (backproject_lds_bytes(p.n_ch, p.block, p.window | 1) > kMaxLds)
            return fail(PL_EUNSUPPORTED, "back-projection staging exceeds the LDS (lower kz_per_lane)");
        p.window_pad = p.window | 1;  // odd row length: conflict-free LDS reads across lanes
    }
    if (p.window > 128)
        return fail(PL_EUNSUPPORTED, "pixels are too coarse for the range grid (window %d > 128)", p.window);
    p.tiles_x = (grid->nx + p.tile_x - 1) / p.tile_x;
    p.tiles_y = (grid->ny + p.tile_y - 1) / p.tile_y;

    // range samples: a multiple of 4 (8-byte stores of split BF16 profiles).
    // The NUFFT's fine grid: for FP32 NUFFT plans the smallest grid of at
    // least 1.25 n_l points, preferring the 64 R sizes (R 2,3,5-smooth, at
    // most 32) of the wavefront-per-pair kernels; other plans keep 2 n_l
    // (2,3,5-smooth; the resampling method's uniform grid and the plan
    // tables use it).
    int nl = static_cast<int>(std::ceil(span / p.du)) + 8;
    nl = std::max(nl, p.window + 2);
    nl = (nl + 3) & ~3;
    const bool nufft32 = p.precision == PL_PREC_FP32 && p.range_method == PL_RANGE_NUFFT;
    if (nufft32) {
        const int want = static_cast<int>(std::ceil(kNufftUpsample * nl));
        int nf = 0;
        for (int r = (want + 63) / 64; r <= 32 && !nf; ++r)
            if (is_fft_friendly(r)) nf = 64 * r;
        if (!nf)
            for (nf = want; !is_fft_friendly(nf); ++nf) {
            }
        p.n_l = nl;
        p.n_fine = nf;
    } else {
        while (!is_fft_friendly(2 * nl)) nl += 4;
        p.n_l = nl;
        p.n_fine = 2 * nl;
    }
    if (p.n_fine > kMaxFine)
        return fail(PL_EUNSUPPORTED, "range grid of %d samples needs a fine grid over %d (lower l_oversample)", p.n_l,
                    kMaxFine);
    factor_radices(p.n_fine, &p.fine_rad);
    if (p.range_method == PL_RANGE_RESAMPLE) {
        // uniform k_L grid whose inverse FFT lands on the range grid: step
        // 2 pi / (n_fine du); a block's band of 2 half_band holds at most
        // n_fine / sigma + 1 of its points, so they never share a bin
        p.dkl = 2.0 * kPi / (p.n_fine * p.du);
        p.k0 = g->k[0];
        p.dk = (g->k[p.n_f - 1] - g->k[0]) / (p.n_f - 1);
        if (!(p.dk > 0) || 2.0 * p.half_band / p.dkl + 2.0 > p.n_fine)
            return fail(PL_EUNSUPPORTED, "resampling grid does not fit the range grid");
        // reference wavenumbers on the grid (the reference cancels between
        // eqs. 8a and 8b, any value is exact): the grid's k' are then whole
        // multiples of dkl and land on FFT bins without a residual shift.  The
        // band edges move by at most dkl / 2 = sigma half_band / n_fine.
        for (int b = 0; b < p.n_blocks; ++b) p.kref[b] = p.dkl * std::nearbyint(p.kref[b] / p.dkl);
    }

    if (int rc = set_spreading(&p, p.sigma_l)) return rc;

    // interpolation weights as cubic polynomials in t = u - floor(u), taps at
    // floor(u) - 1 .. floor(u) + 2
    static const float bsp[4][4] = {{1.f / 6, -0.5f, 0.5f, -1.f / 6},
                                    {4.f / 6, 0.f, -1.f, 0.5f},
                                    {1.f / 6, 0.5f, 0.5f, -0.5f},
                                    {0.f, 0.f, 0.f, 1.f / 6}};
    static const float lag[4][4] = {{0.f, -1.f / 3, 0.5f, -1.f / 6},
                                    {1.f, -0.5f, -1.f, 0.5f},
                                    {0.f, 1.f, 0.5f, -0.5f},
                                    {0.f, -1.f / 6, 0.f, 1.f / 6}};
    static const float lin[4][4] = {{0.f, 0.f, 0.f, 0.f}, {1.f, -1.f, 0.f, 0.f}, {0.f, 1.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    const float(*src)[4] = p.interp == PL_INTERP_BSPLINE4 ? bsp : (p.interp == PL_INTERP_LAGRANGE4 ? lag : lin);
    std::memcpy(p.coef, src, sizeof(p.coef));

    if (int rc = set_layout(&p)) return rc;
    p.need = p.total;
    *out = p;
    return PL_OK;
}

int make_call_plan(const pl_geometry* g, const pl_image_grid* grid, const pl_hybrid_opts* opts, bool own_workspace,
                   HybridPlan* out) {
    if (int rc = make_plan(g, grid, opts, out)) return rc;
    // The BF16 and FP16 modes with split operands (or the vector
    // back-projection) take the window form of their FP32 plan: it is the
    // more accurate and the faster one (256 k_z x 320 channels x 200x200
    // pixels: 0.92 against 1.49 ms), from some 64x64 pixels on: at 44x44 its
    // range compression costs what its back-projection gains (182 against
    // 175 us; 48x77 and 68x87 even).
    HybridPlan base = *out, w;
    if (out->precision != PL_PREC_FP32) {
        if ((out->force_bp_mfma != 0 && out->force_bp_mfma != 1) || out->nx * static_cast<long long>(out->ny) < 4096)
            return PL_OK;
        pl_hybrid_opts o = *opts;
        o.precision = PL_PREC_FP32;
        o.mfma_backprojection = 0;
        if (make_plan(g, grid, &o, &base)) {
            clear_error();
            return PL_OK;
        }
    }
    if (window_plan(g, grid, base, *out, own_workspace, &w)) {
        w.need = std::max(w.total, out->total);
        *out = w;
    }
    return PL_OK;
}

// The key is compared byte by byte, so it must hold no padding.
static_assert(sizeof(pl_image_grid) == 2 * sizeof(int32_t) + 4 * sizeof(double), "padding in pl_image_grid");
static_assert(sizeof(pl_hybrid_opts) == 10 * sizeof(int32_t) + 2 * sizeof(double), "padding in pl_hybrid_opts");

int cached_plan(const pl_geometry* g, const pl_image_grid* grid, const pl_hybrid_opts* opts, PlanUse use,
                HybridPlan* out) {
    auto plan = [&] {
        return use == PlanUse::kSteps ? make_plan(g, grid, opts, out)
                                      : make_call_plan(g, grid, opts, use == PlanUse::kCallAlone, out);
    };
    if (!g || !grid || !out) return plan();                         // its error
    const pl_hybrid_opts key = opts ? *opts : pl_hybrid_opts{};     // no options: all zero
    {
        std::lock_guard<std::mutex> lock(g->plan_mu);
        for (const auto& c : g->plans)
            if (c.use == use && !std::memcmp(&c.grid, grid, sizeof(*grid)) &&
                !std::memcmp(&c.opts, &key, sizeof(key))) {
                *out = c.plan;
                return PL_OK;
            }
    }
    if (int rc = plan()) return rc;   // outside the lock; errors are not kept
    std::lock_guard<std::mutex> lock(g->plan_mu);
    if (g->plans.size() < pl_geometry::kPlanCache) {
        g->plans.push_back({*grid, key, use, *out});
    } else {
        g->plans[g->next_plan] = {*grid, key, use, *out};
        g->next_plan = (g->next_plan + 1) % pl_geometry::kPlanCache;
    }
    return PL_OK;
}

}  // namespace pl
