// Test-only shim: exposes the packer of the quotient kernels
// (quotient_tables.cpp) to the CPU tests.  Built with g++ by the tests.
#include <cstring>
#include <string>

#include "quotient.hpp"

extern "C" {

int qt_chunk(int n_vars, int max_exp, int pad, int64_t max_m, int words)
{
    return pe::quot_chunk(n_vars, max_exp, pad != 0, max_m, words);
}

int64_t qt_lds(int n_vars, int max_exp, int pad, int CH, int multi, int nbuf, int words)
{
    return (int64_t)pe::quot_lds_bytes(n_vars, max_exp, pad != 0, CH, multi != 0, nbuf, words);
}

int qt_point_exp(int d) { return pe::quot_point_exp(d); }

void *qt_build(int32_t n_vars, int32_t n_polys, int64_t n_monos, const int64_t *ps, const int64_t *ms,
               const int32_t *pos, const int32_t *exp, int CH, int *pad, int64_t *max_m)
{
    auto *t = new pe::QuotTables();
    t->CH = CH;
    pe::CsrView v{n_vars, n_polys, n_monos, ps, ms, pos, exp};
    pe::quot_shape(v, t->pad, *max_m);
    *pad = t->pad;
    if (!pe::build_quot_tables(v, *t).empty()) {
        delete t;
        return nullptr;
    }
    return t;
}

void qt_free(void *p) { delete static_cast<pe::QuotTables *>(p); }

// table `which` copied to dst (when given); returns its number of entries
int64_t qt_table(void *p, int which, void *dst)
{
    auto *t = static_cast<pe::QuotTables *>(p);
    auto give = [&](const auto &v) {
        if (dst) std::memcpy(dst, v.data(), v.size() * sizeof(v[0]));
        return (int64_t)v.size();
    };
    switch (which) {
    case 0: return give(t->words);
    case 1: return give(t->mono);
    case 2: return give(t->slice);
    case 3: return give(t->chunk);
    case 4: return give(t->poly);
    case 5: return give(t->block);
    case 6: return give(t->runs);
    case 7: return give(t->out);
    case 8: return t->n_blk;
    default: return t->multi ? 1 : 0;
    }
}

}  // extern "C"
