// The library's series (csrc/moment_series.h) behind a C function, for tests/test_moment_series.py.
#include "moment_series.h"

extern "C" void series(int kernel, double delta, double sigma, double trunc, double nu, int exact, int* terms, float* edge,
                       float* coef) {
    ra_sampling s{};
    s.c = delta;
    s.fs = 1.0;
    s.K = 1;
    s.sigma = sigma;
    s.trunc = trunc;
    s.kernel = kernel;
    s.nu = nu;
    MomSeries m;
    make_series(&s, exact != 0, m);
    const MomTerms& t = m.terms;
    const int v[5] = {t.fwd, t.vol, t.pose, t.xkind, t.flip != 0u};
    std::memcpy(terms, v, sizeof(v));
    const float e[6] = {t.thr, t.ev[0], t.ev[1], t.ev[2], t.ev[3], t.kx};
    std::memcpy(edge, e, sizeof(e));
    const MomCoef* of[3] = {&m.fwd, &m.vol, &m.pose};
    for (int i = 0; i < 3; ++i)
        if (v[i]) std::memcpy(coef + i * (JMAX + 1) * MOM_MAX, of[i]->d, sizeof(MomCoef));
}
