// Test-only shim: the complex reciprocals of dd.hpp, compiled for the host.
#include "dd.hpp"

using namespace pe;

extern "C" {
// b, o: re hi, re lo, im hi, im lo
void rp_dd(const double *b, double *o)
{
    const ArithDD::C r = ArithDD::recip({{b[0], b[1]}, {b[2], b[3]}});
    o[0] = r.re.hi;
    o[1] = r.re.lo;
    o[2] = r.im.hi;
    o[3] = r.im.lo;
}
void rp_f64(const double *b, double *o)
{
    const Arith64::C r = Arith64::recip({b[0], b[1]});
    o[0] = r.re;
    o[1] = r.im;
}
}
