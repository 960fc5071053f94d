// Host-side driver of the rate quadrature's sum (test infrastructure).
#include "../../paper_1606_02862_amd/csrc/ionize_internal.hpp"

extern "C" void rsh_sum(int64_t n, const double* r, const double* b, const double* c, const double* rule64, double* one,
                        double* plain)
{
    static pic::GlRule rule;
    for (int k = 0; k < pic::GL_NODES; ++k) {
        rule.x[k] = rule64[k];
        rule.w[k] = rule64[pic::GL_NODES + k];
    }
    pic::log_table(reinterpret_cast<double*>(rule.lt));
    for (int64_t i = 0; i < n; ++i) {
        one[i] = pic::lotz_sum4(r[i], b[i], c[i], rule);
        double s = 0.0;  // one chain over all nodes, library logarithm
        for (int k = 0; k < pic::GL_NODES; ++k) {
            const double xr = rule.x[k] * r[i];
            s = fma(rule.w[k] * log1p(xr), 1.0 - b[i] * exp(-c[i] * xr), s);
        }
        plain[i] = s;
    }
}
