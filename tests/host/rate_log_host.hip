// Host-side driver of the rate quadrature's logarithm (test infrastructure).
#include "../../paper_1606_02862_amd/csrc/rate_log.hpp"

extern "C" void rlh_log1p(int64_t n, const double* y, double* out)
{
    double2 tab[pic::LOG_N];
    pic::log_table(reinterpret_cast<double*>(tab));
    for (int64_t i = 0; i < n; ++i) out[i] = pic::log1p_pos(y[i], tab);
}
