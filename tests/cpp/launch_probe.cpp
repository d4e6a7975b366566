// Test-only shim: the host functions that choose and size the launches of the
// quotient kernels (quotient_tables.cpp, launch_limits.hpp).  Built with g++ by the tests.
#include "launch_limits.hpp"
#include "quotient.hpp"

extern "C" {

int lp_chunk(int n_vars, int max_exp, int pad, int64_t max_m, int words)
{
    return pe::quot_chunk(n_vars, max_exp, pad != 0, max_m, words);
}

int64_t lp_lds(int n_vars, int max_exp, int pad, int CH, int multi, int nbuf, int words)
{
    return (int64_t)pe::quot_lds_bytes(n_vars, max_exp, pad != 0, CH, multi != 0, nbuf, words);
}

int64_t lp_small_lds(int64_t general, int64_t quot) { return (int64_t)pe::small_lds_bytes(general, quot); }

int lp_single(int64_t units, int64_t general, int64_t quot)
{
    return pe::single_launch(units, pe::kSmallUnits, general, quot);
}

int64_t lp_single_units(int n_vars, int max_k, int64_t max_m, int words, int jac)
{
    return pe::single_launch_units(n_vars, max_k, max_m, words, jac != 0);
}

int64_t lp_add_skip_words(int64_t lds)
{
    size_t v = (size_t)lds;
    return pe::add_skip_words(v) ? (int64_t)v : -1;
}

int lp_window(int d, int *check)
{
    bool c;
    const int b = pe::quot_window(d, c);
    *check = c;
    return b;
}

int lp_coef_ok(const double *c) { return pe::quot_coef_ok(c[0], c[1], c[2], c[3]); }

int64_t lp_max_workgroups(int threads) { return pe::max_workgroups(threads); }

int64_t lp_strided_grid(int64_t work, int threads) { return pe::strided_grid(work, threads); }

}  // extern "C"
