// moment_series.h -- the series of the moment forms, made on the host in FP64: a pair's window as polynomials in its
// offset t from its nearest sample, in units of half a sample (see "forward in moment form" in radiate.hip).
#pragma once

#include <algorithm>
#include <cmath>
#include <cstring>

#include "radiate.h"

constexpr int JMAX = 40;              // largest supported window half-width in samples
constexpr int MOM_MAX = 12;           // largest number of moments
constexpr int MOM_G = 8;              // and the Gaussian's
constexpr double FM_TOL = 2e-7;       // largest admitted expansion error, relative to the peak
constexpr double FM_EDGE = 0.004;     // largest phi at the window's edge (other profiles), relative to the peak
constexpr double AM_TOL = 2.5e-8;     // that error where the series' derivative is used (its 8 terms' grows 8-fold in rms)
constexpr double WIDE_GAUSS = 0.559;  // delta/sigma up to which Gaussian adjoints take the rows whole for any window, and a table of any size

struct MomCoef {
    float d[(JMAX + 1) * MOM_MAX];     // D_n(j) / delta at j * MOM_MAX + n, j >= 0; D_n(-j) = (-1)^(n+1) D_n(j)
};

// Terms of the moment forms' series (0: the form cannot be taken).
struct MomTerms {
    int fwd, vol, pose;
    float thr, ev[4], es, kx;      // Geo's of the same names
    unsigned flip;
    int xkind;
};

struct MomSeries {
    double key[4] = {0.0, 0.0, 0.0, 0.0};  // profile, delta / width, window, nu
    MomTerms terms{};
    MomCoef fwd, vol, pose;                // with the terms of the forward, of dL/dp0 alone and of the element gradients
};

// phi(x delta) / delta of a source profile, x in samples, dd = delta / w.
inline double profile(const ra_sampling* samp, double dd, double x) {
    const double y = std::fabs(x) * dd;
    switch (samp->kernel) {
        case RA_KERNEL_EXPONENTIAL: return x * std::exp(-y);
        case RA_KERNEL_POWER: return x * std::pow(1.0 + y * y, -samp->nu);
        case RA_KERNEL_UNIFORM: return x;
        default: return x * std::exp(-0.5 * y * y);
    }
}

// Chebyshev coefficients in t of phi((t/2 - j) delta) / delta for j = j0..j1, from MOM_NODES nodes; tail[n] bounds
// what is cut after n terms, relative to `peak`.
constexpr int MOM_NODES = 24;

inline void mom_series(const ra_sampling* samp, double dd, int j0, int j1, double peak, double cheb[MOM_MAX][JMAX + 1],
                       double tail[MOM_MAX + 1]) {
    struct Nodes {
        double c[MOM_NODES][MOM_NODES];
        Nodes() {
            for (int k = 0; k < MOM_NODES; ++k)
                for (int i = 0; i < MOM_NODES; ++i) c[k][i] = std::cos(3.14159265358979323846 * k * (i + 0.5) / MOM_NODES);
        }
    };
    static const Nodes nodes;
    const double(&cs)[MOM_NODES][MOM_NODES] = nodes.c;
    for (int n = 0; n <= MOM_MAX; ++n) tail[n] = 0.0;
    for (int j = j0; j <= j1; ++j) {
        double f[MOM_NODES];
        for (int i = 0; i < MOM_NODES; ++i) f[i] = profile(samp, dd, 0.5 * cs[1][i] - j);
        double rest = 0.0;
        for (int k = MOM_NODES - 1; k >= 0; --k) {
            double c = 0.0;
            for (int i = 0; i < MOM_NODES; ++i) c += f[i] * cs[k][i];
            c *= (k ? 2.0 : 1.0) / MOM_NODES;
            if (k < MOM_MAX) cheb[k][j] = c;
            rest += std::fabs(c);
            if (k <= MOM_MAX) tail[k] = std::max(tail[k], rest / peak);
        }
    }
}

// The sum of the first nm Chebyshev terms of sample j as a polynomial in t.
inline void mom_monomials(const double cheb[MOM_MAX][JMAX + 1], int nm, int j, float* out) {
    double T[MOM_MAX][MOM_MAX] = {};                       // T[k][n]: coefficient of t^n in T_k
    T[0][0] = 1.0;
    T[1][1] = 1.0;
    for (int k = 2; k < nm; ++k)
        for (int n = 0; n < nm; ++n) T[k][n] = (n ? 2.0 * T[k - 1][n - 1] : 0.0) - T[k - 2][n];
    for (int n = 0; n < nm; ++n) {
        double v = 0.0;
        for (int k = n; k < nm; ++k) v += cheb[k][j] * T[k][n];
        out[n] = (float)v;
    }
}

// The moment forms' series for a sampling; `exact`: the Gaussian's row forms take this window whole.  Their numbers of
// terms are the fewest of those compiled whose cut series is within FM_TOL (AM_TOL where the derivative is used too):
//   Gaussian     6 up to delta/sigma 0.41, 7 up to 0.64, 8 up to 1.11 (the row form's own rounding is about 4e-7); 8 with
//                derivatives, up to 0.74.  The window's rows are taken whole, as the Gaussian's row forms do for
//                the half-widths of RA_EXACT_LIST; for longer windows those test each term, so the form is taken
//                there only from 6 sigma on, where the terms in question are below 1.5e-7 of the peak.
//   the others   6 or 8 for the exponential (without the centre sample, which is added by itself), 8 to 12 for the
//                power law.  A sample that is in the window for some offsets only is added by itself too, by its
//                first four terms.  Only where phi has fallen to FM_EDGE of its peak at the window's edge: on
//                which side a pair within rounding of the edge falls is not what the row forms or FP64 say, and
//                moves a result by one term's edge value (by 1.4e-3 of the rms at an edge value of 0.0135).
//                The uniform sphere keeps the row forms always; a power law with nu = 2 passes from 9.1
//                widths on, the exponential from 8.7.
inline void make_series(const ra_sampling* samp, bool exact, MomSeries& m) {
    const double delta = samp->c / samp->fs, dd = delta / samp->sigma, jw = samp->trunc * samp->sigma / delta;
    MomTerms& t = m.terms;
    t = MomTerms{};
    const int jo = (int)std::floor(jw + 0.5), kt = samp->kernel;
    if (jo < 1 || jo > JMAX || kt == RA_KERNEL_UNIFORM || (kt == RA_KERNEL_GAUSSIAN && !(exact || samp->trunc >= 6.0))) return;
    // phi's peak: at the width (power law: width / sqrt(2 nu - 1)), or the window's edge before it
    const double top = std::min(jw, (kt == RA_KERNEL_POWER ? 1.0 / std::sqrt(2.0 * samp->nu - 1.0) : 1.0) / dd);
    const double peak = profile(samp, dd, top);
    double cheb[MOM_MAX][JMAX + 1] = {}, ce[MOM_MAX][JMAX + 1] = {}, te[MOM_MAX + 1];
    const double edge = 2.0 * (jo - jw);                   // kc + jo is in the window for t >= edge
    const int j0 = kt == RA_KERNEL_EXPONENTIAL ? 1 : 0, j1 = kt == RA_KERNEL_GAUSSIAN || edge <= 0.0 ? jo : jo - 1;
    double tail[MOM_MAX + 1];
    mom_series(samp, dd, j0, j1, peak, cheb, tail);
    if (kt != RA_KERNEL_GAUSSIAN) {
        mom_series(samp, dd, jo, jo, peak, ce, te);
        if (!(te[4] <= FM_TOL) || profile(samp, dd, jw) > FM_EDGE * peak) return;
        t.xkind = kt == RA_KERNEL_EXPONENTIAL ? 2 : 1;
        mom_monomials(ce, 4, jo, t.ev);
        t.thr = (float)edge;
        if (edge <= 0.0) {                                 // take back phi at kc - jo for t > -edge: F(|t|) = E(-|t|)
            t.thr = std::nextafterf((float)-edge, 2.0f);
            t.flip = 0x80000000u;
            t.ev[1] = -t.ev[1];
            t.ev[3] = -t.ev[3];
        }
        // |phi| / delta of the single samples: three of them meet in a row at most (centre, kc + jt, kc - jt)
        double top = 0.0;
        for (int i = -1; i <= 1; ++i) top = std::max(top, std::fabs(profile(samp, dd, 0.5 * i - jo)));
        t.es = (float)(1.0 / (0.5 + 2.0 * std::max(top, peak)));
        t.kx = (float)(-0.5 * dd * 1.4426950408889634);
    }
    static const int terms[3][3] = {{6, 7, 8}, {6, 8, 8}, {8, 10, 12}};      // by profile
    auto fewest = [&](double tol, int from) {
        for (int i = from; i < 3; ++i)
            if (tail[terms[kt][i]] <= tol) return terms[kt][i];
        return 0;
    };
    t.fwd = fewest(FM_TOL, 0);
    if (!t.fwd) return;
    t.vol = kt == RA_KERNEL_GAUSSIAN ? t.fwd : kt == RA_KERNEL_POWER && t.fwd > 8 ? 12 : terms[kt][1] == 10 ? 8 : terms[kt][1];
    t.pose = kt == RA_KERNEL_POWER ? (tail[8] <= AM_TOL ? 8 : fewest(AM_TOL, 2)) : fewest(AM_TOL, 2);
    // Short windows of narrow Gaussians: the adjoints' row forms test the window's outermost samples, whose terms
    // are psi(trunc) of the peak (1.5e-7 from 6 sigma on, 1.6e-3 at 4)
    if (kt == RA_KERNEL_GAUSSIAN && samp->trunc < 6.0 && dd > WIDE_GAUSS) t.vol = t.pose = 0;
    const int nm[3] = {t.fwd, t.vol, t.pose};
    MomCoef* const out[3] = {&m.fwd, &m.vol, &m.pose};
    for (int i = 0; i < 3; ++i) {
        std::memset(out[i], 0, sizeof(MomCoef));
        for (int j = j0; nm[i] && j <= j1; ++j) mom_monomials(cheb, nm[i], j, out[i]->d + j * MOM_MAX);
    }
}
