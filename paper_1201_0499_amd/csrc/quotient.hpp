// Evaluation with the Jacobian by quotients: tables, launch arguments and
// launch wrappers (kernels in quotient.hip, packing in quotient_tables.cpp).
//
// With V_s = c_s x^{a_s} the value of monomial s (Section 2, equation (1)),
//
//     f_p = sum_s V_s,     df_p/dx_i = (1 / x_i) sum_s a_{s,i} V_s,
//
// so a monomial of k variables costs k products for its value and one scaled
// addition per variable, where the forward and backward products of
// Section 3.2 with their common factor cost about 5k products.  The quotient
// exists only for x_i != 0, and the products must stay away from overflow
// and underflow; see the rules below.  Whatever they refuse goes to the
// general kernel (eval.hip), which has no such restriction.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <string>
#include <vector>

#include "schedule.hpp"

namespace pe {

// Factors x_i^{a_i} of a monomial are multiplied in quads.  The canonical
// order of a monomial's product (and so every bit of it) does not depend on
// how many lanes take part: its quads fall into kParts contiguous ranges,
// each range is multiplied from the left, then (r0 r1)(r2 r3).  A run of
// terms is added in kParts interleaved partial sums, combined the same way.
constexpr int kQuad = 4;
constexpr int kParts = 4;
// Outputs of a chunk are summed in blocks of kRankBlock ranks (by run
// length), padded to the longest run of the block.
constexpr int kRankBlock = 16;
// An entry of a run: position of the monomial's value in the chunk in the
// low kEntryBits bits, the exponent above them; padding has exponent 0.
constexpr int kEntryBits = 11;
constexpr int kMaxQuotExp = (1 << (16 - kEntryBits)) - 1;
constexpr int kMaxQuotChunk = 1024;  // monomials per chunk, at most (<= 2^kEntryBits)

// Range rules.  Partial products of a monomial (quads of factors apart) must
// have a binary exponent within +-kProductExp, which the kernel checks.  A quad
// of factors is bounded by the same: by the points, where that leaves them a
// window of at least 2^+-kWideExp, so that a single quad passes the check
// wherever it is made; else by checking quads too, and then the points only
// keep the power table's entries within 2^+-kPowerExp (quot_window).  Either
// way what is refused does not depend on how many lanes share a monomial.
// (Products of two factors are within 2^+-600 there; those of quads may
// overflow or vanish, and are then out of range.)  With coefficients within
// 2^+-kCoefExp (or zero) no product that counts, nor an error term of
// quad-double arithmetic, overflows or becomes subnormal: the smallest entry of
// J is 2^-(400 + 300 + 60), its error terms 2^-212 of it.
constexpr int kWideExp = 16;
constexpr int kPowerExp = 300;
constexpr int kProductExp = 400;
constexpr int kCoefExp = 300;

// Whether the quotient kernels take a coefficient (its parts as double-words):
// its larger part within 2^+-kCoefExp, or zero; finite, as a NaN would be refused
// at every point, after the work.
inline bool quot_coef_ok(double re_hi, double re_lo, double im_hi, double im_lo)
{
    if (!std::isfinite(re_hi) || !std::isfinite(re_lo) || !std::isfinite(im_hi) || !std::isfinite(im_lo)) return false;
    const double big = std::max(std::fabs(re_hi), std::fabs(im_hi));
    return big == 0.0 ? re_lo == 0.0 && im_lo == 0.0 : std::abs(std::ilogb(big)) < kCoefExp;
}

// Largest binary exponent of a coordinate (either sign) for maximal exponent
// d: kQuad factors of at most 2^(d (b + 1/2)) each stay within 2^kProductExp.
inline int quot_point_exp(int d)
{
    const int b = (2 * kProductExp / kQuad - d) / (2 * d);
    return b < 0 ? 0 : (b > 60 ? 60 : b);
}

// The window of the points for maximal exponent d: the larger part of every
// coordinate has a binary exponent of at most b, either sign.  Up to d = 5 a
// window of 2^+-18 or more comes without checked quads, above 2^+-48 (d = 6) to
// 2^+-8 (d = 31) with them; without them it would be 2^+-8 at d = 10 and 2^+-1
// at d = 31, where complex Gaussian coordinates leave 9 polynomials in 10 to the
// general kernel (n = 64, m = 128, k = 16, 200 points in double-double, which
// that kernel alone takes 669 us for: 874 us without, 312 us with).
inline int quot_window(int d, bool &check_quads)
{
    const int b = quot_point_exp(d) - 1;
    check_quads = b < kWideExp;
    if (!check_quads) return b;
    const int c = (2 * kPowerExp - d) / (2 * d);
    return std::min(c, 60) - 1;
}

// Packed tables of one system for chunks of CH monomials.  Monomials of a
// polynomial are ordered by their number of variables, most first (stable),
// so that the 64 monomials of a slice need about the same number of quads;
// one constant monomial per polynomial is folded into the value output.  The
// order of a monomial's factors and of a run's terms is chosen for the LDS
// (quotient_tables.cpp).
struct QuotTables {
    int CH = 0;            // monomials per chunk (a multiple of 64)
    int n_blk = 0;         // rank blocks per chunk
    bool pad = true;       // the power table has an entry 1 for incomplete quads (set by
                           //   the caller; may be false if every monomial but the
                           //   folded ones has the same number of variables, a
                           //   multiple of kQuad)
    bool multi = false;    // some polynomial has more than one chunk
    bool complete = false; // every variable occurs in some polynomial (see poly)
    int n_chunks = 0;
    std::vector<uint16_t> words;     // per slice [quads][monomials][kQuad]: power-table
                                     //   entry (a-1) n + variable, or d n: the entry 1
    std::vector<int32_t> mono;       // [monomials in table order]: index in the system
    std::vector<int32_t> slice;      // [slices][2]: first quad in words, quads
    std::vector<int32_t> chunk;      // [chunks][4]: first monomial (table order),
                                     //   monomials, first slice, first rank block
    std::vector<int32_t> poly;       // [n_polys][4]: first chunk, end chunk, 1 + index
                                     //   of the folded constant (0: none), 1 if every
                                     //   variable occurs in it
    std::vector<int32_t> block;      // [chunks][n_blk][2]: first row, rows
    std::vector<uint16_t> runs;      // [rows][kRankBlock][kParts] entries
    std::vector<uint16_t> out;       // [chunks][n_blk * kRankBlock]: output of a rank
                                     //   (0xFFFF past the last)
};

// Monomials per chunk for values of `words` doubles: what one workgroup's
// LDS holds, at most kMaxQuotChunk; 0 if the power table leaves no room or
// the system is outside the packing (exponents, variables).
int quot_chunk(int n_vars, int max_exp, bool pad, int64_t max_m, int words);

// LDS bytes of a workgroup with nbuf buffers of chunk values.
size_t quot_lds_bytes(int n_vars, int max_exp, bool pad, int CH, bool multi, int nbuf, int words);

// Words for a workgroup's waves: whether the wave saw a coordinate out of range
// (see quot_table); after the tables, where there is one buffer of values.
constexpr size_t kQuotWordBytes = 64;
// Where they fit a workgroup's `lds` bytes and leave as many workgroups on a
// CU, add_skip_words adds them.
bool add_skip_words(size_t &lds);
// Calls of at most this many (polynomial, point) pairs run in one launch
// (small.hip): five workgroups per CU.  One MI355X, two launches against one:
// n = 350, m = 69, k = 8, 3 points in FP64 17.5 and 14.7 us, n = 16, m = 64, k
// = 16, 128 points (2048 pairs) 17 and 18.3 us.  With the Jacobian, where most
// outputs of many have no or one term, so that the table and the stores are
// the work, up to kSparseUnits pairs (two launches against one): double-double,
// n = 400, m = 8, k = 2, 5 points 36.5 and 28.3 us, 35 points 161 and 151 us, n
// = 300, m = 200, k = 2, 23 points 94 and 82 us, n = 128, m = 8, k = 2, 20
// points 27 and 23 us, n = 300, m = 60, k = 4, 8 points 41 and 36 us; FP64, n =
// 400, m = 8, k = 2, 35 points 89 and 71 us, m = 60, k = 6, 5 points 26 and 19
// us, n = 500, m = 60, k = 12, 3 points 24 and 20 us; but n = 300, m = 60, k = 6,
// 13 points in double-double 56 and 69 us, and n = 128, m = 8, k = 2, 54 points
// 41 and 53 us.
constexpr int64_t kSmallUnits = 1280;
constexpr int64_t kSparseUnits = 16384;
int64_t single_launch_units(int n_vars, int max_k, int64_t max_m, int words, bool jac);
// ... whose workgroups hold the general stages' LDS (general_lds bytes), or
// the quotients' (quot_lds, for one point and one buffer) and then a flag.
constexpr size_t kSmallFlagBytes = 16 + kQuotWordBytes;
size_t small_lds_bytes(size_t general_lds, size_t quot_lds);
// Whether a call of `units` pairs, of at most `most`, runs in one launch.
// Tables of the quotients may fill the LDS without the flag (n = 512, m = 512,
// d = 8 in double-double): two launches then, whatever the number of pairs.
bool single_launch(int64_t units, int64_t most, size_t general_lds, size_t quot_lds);

// Whether the power table needs the entry 1 (see QuotTables::pad), and the
// most monomials of a polynomial without its folded constant.
void quot_shape(const CsrView &S, bool &pad, int64_t &max_m);

// Fill t for chunks of t.CH monomials; empty string on success.
std::string build_quot_tables(const CsrView &S, QuotTables &t);

}  // namespace pe
