// Host-side packing for the quotient kernels.  See quotient.hpp.
#include "quotient.hpp"

#include <algorithm>
#include <climits>

#include "lds_budget.hpp"

namespace pe {

size_t quot_lds_bytes(int n_vars, int max_exp, bool pad, int CH, bool multi, int nbuf, int words)
{
    const size_t n = (size_t)n_vars;
    const size_t values =
        (size_t)max_exp * n + (pad ? 1 : 0) + n + (size_t)nbuf * (size_t)CH + (multi ? n + 1 : 0);
    return values * (size_t)words * sizeof(double);
}

bool add_skip_words(size_t &lds)
{
    const size_t with = lds + kQuotWordBytes;
    if (with > kLdsBytes || kLdsBytes / with < kLdsBytes / lds) return false;
    lds = with;
    return true;
}

size_t small_lds_bytes(size_t general_lds, size_t quot_lds)
{
    return std::max(general_lds, quot_lds + kSmallFlagBytes);
}

int64_t single_launch_units(int n_vars, int max_k, int64_t max_m, int words, bool jac)
{
    const int64_t terms = max_m * max_k;
    if (!jac || words == 8 || n_vars < 100) return kSmallUnits;
    if (max_k <= 2) {
        const bool less = n_vars < 200 || (words == 4 && n_vars >= 450 && 2 * terms >= n_vars);
        return less ? kSparseUnits / 4 : kSparseUnits;
    }
    if (n_vars < 200) return kSmallUnits;
    if (4 * terms <= n_vars) return kSparseUnits;
    const bool few = 2 * terms <= n_vars || (n_vars >= 300 && terms <= n_vars) || (n_vars >= 400 && terms < 2 * n_vars);
    return few ? kSparseUnits / 4 : kSmallUnits;
}

bool single_launch(int64_t units, int64_t most, size_t general_lds, size_t quot_lds)
{
    return units <= most && small_lds_bytes(general_lds, quot_lds) <= kLdsBytes;
}

int quot_chunk(int n_vars, int max_exp, bool pad, int64_t max_m, int words)
{
    if (max_exp > kMaxQuotExp || n_vars >= 0xFFFF || (int64_t)max_exp * n_vars >= 0xFFFF ||
        quot_point_exp(max_exp) < 2)
        return 0;
    const int64_t whole = (std::max<int64_t>(1, max_m) + 63) / 64 * 64;
    int ch = (int)std::min<int64_t>(whole, kMaxQuotChunk);
    // equal chunks rather than full ones and a short last one
    const int64_t parts = (whole + ch - 1) / ch;
    ch = (int)((whole / 64 + parts - 1) / parts * 64);
    for (; ch >= 64; ch -= 64)
        if (quot_lds_bytes(n_vars, max_exp, pad, ch, ch < max_m, 1, words) <= kLdsBytes) return ch;
    return 0;
}

void quot_shape(const CsrView &S, bool &pad, int64_t &max_m)
{
    pad = false;
    max_m = 0;
    int64_t kmax = 0;
    for (int64_t s = 0; s < S.n_monos; ++s) kmax = std::max(kmax, S.mono_start[s + 1] - S.mono_start[s]);
    if (kmax % kQuad) pad = true;
    for (int p = 0; p < S.n_polys; ++p) {
        int64_t constants = 0;
        for (int64_t s = S.poly_start[p]; s < S.poly_start[p + 1]; ++s) {
            const int64_t k = S.mono_start[s + 1] - S.mono_start[s];
            if (k == 0)
                ++constants;
            else if (k != kmax)
                pad = true;
        }
        if (constants > 1) pad = true;  // only one is folded
        max_m = std::max(max_m, S.poly_start[p + 1] - S.poly_start[p] - (constants > 0 ? 1 : 0));
    }
}

namespace {

// LDS reads of 16 bytes per lane serve 16 consecutive lanes at a time, each
// from its own sixteenth of the banks (entry modulo 16) at best; random
// entries need three times as long (3.1 lanes on the worst sixteenth).  The
// order of a monomial's factors and of a run's terms is free, so the packer
// chooses it: a pool holds one lane's entries by bank, and each step of 16
// lanes takes one from each, on banks not yet used where there are such.
struct Pool {
    std::vector<uint16_t> item;  // the entries, by bank
    int next[17];                // next[b] .. end of bank b in item
    int left[16];                // entries left on each bank
    unsigned mask = 0;           // banks with entries left
    int total = 0;               // entries left

    template <class Bank>
    void fill(const uint16_t *src, int n, const Bank &bank)
    {
        std::fill(left, left + 16, 0);
        for (int i = 0; i < n; ++i) ++left[bank(src[i])];
        next[0] = 0;
        mask = 0;
        for (int b = 0; b < 16; ++b) {
            next[b + 1] = next[b] + left[b];
            if (left[b]) mask |= 1u << b;
        }
        item.resize((size_t)n);
        int at[16];
        std::copy(next, next + 16, at);
        for (int i = 0; i < n; ++i) item[(size_t)at[bank(src[i])]++] = src[i];
        total = n;
    }
    uint16_t pop(int b) { return item[(size_t)next[b]++]; }
    void reserve(int b)
    {
        if (--left[b] == 0) mask &= ~(1u << b);
        --total;
    }
    void give_back(int b)
    {
        ++left[b];
        mask |= 1u << b;
        ++total;
    }
};

// One step: a bank for each of `lanes` lanes (of pool lane_pool[l]; -1: the
// pool is empty), distinct if that is easy: a lane without a free bank may
// take another's if that one finds a free one instead.
void choose_banks(Pool *const *lane_pool, int lanes, int (&bank)[16])
{
    unsigned free = 0xFFFFu;
    int owner[16];
    for (int l = 0; l < lanes; ++l) {
        Pool &me = *lane_pool[l];
        if (me.total == 0) {
            bank[l] = -1;
            continue;
        }
        int b = -1;
        if (me.mask & free) {
            b = __builtin_ctz(me.mask & free);
        } else {
            for (unsigned m = me.mask; m; m &= m - 1) {
                const int c = __builtin_ctz(m), o = owner[c];
                const unsigned other = lane_pool[o]->mask & free;
                if (!other) continue;
                const int d = __builtin_ctz(other);
                lane_pool[o]->give_back(c);
                lane_pool[o]->reserve(d);
                bank[o] = d;
                owner[d] = o;
                free &= ~(1u << d);
                b = c;
                break;
            }
            if (b < 0) b = __builtin_ctz(me.mask);
        }
        me.reserve(b);
        bank[l] = b;
        owner[b] = l;
        free &= ~(1u << b);
    }
}

}  // namespace

std::string build_quot_tables(const CsrView &S, QuotTables &t)
{
    const int n = S.n_vars, CH = t.CH;
    if (CH < 64 || CH % 64 || CH > kMaxQuotChunk) return "invalid chunk";
    if (S.n_monos >= (int64_t)INT32_MAX) return "too many monomials";
    t.n_blk = (n + kRankBlock - 1) / kRankBlock;
    const int n_rank = t.n_blk * kRankBlock;
    int max_exp = 1;
    for (int64_t e = 0; e < (S.n_monos ? S.mono_start[S.n_monos] : 0); ++e) max_exp = std::max(max_exp, S.exp[e]);
    if (max_exp > kMaxQuotExp) return "exponents too large";
    t.multi = t.complete = false;
    t.words.clear();
    t.mono.clear();
    t.slice.clear();
    t.chunk.clear();
    t.poly.clear();
    t.block.clear();
    t.runs.clear();
    t.out.clear();
    t.mono.reserve((size_t)S.n_monos);
    std::vector<int32_t> len((size_t)n), rank((size_t)n), at((size_t)n + 1), order((size_t)n), bin;
    std::vector<char> has((size_t)n);
    std::vector<int32_t> by_k[257];
    Pool pool[kRankBlock];
    std::vector<uint16_t> list, terms;
    std::vector<int32_t> first_term;
    const uint16_t pad_word = (uint16_t)(max_exp * n);
    int64_t rows_total = 0;
    for (int p = 0; p < S.n_polys; ++p) {
        const int64_t s0 = S.poly_start[p], s1 = S.poly_start[p + 1];
        int32_t fold = 0;
        int kmax = 0;
        for (int64_t s = s0; s < s1; ++s) {
            const int k = (int)(S.mono_start[s + 1] - S.mono_start[s]);
            if (k > 256) return "a monomial has more than 256 variables";
            if (k == 0) fold = (int32_t)s + 1;  // the last one
            kmax = std::max(kmax, k);
            by_k[k].push_back((int32_t)s);
        }
        const int64_t first = (int64_t)t.mono.size();
        for (int k = kmax; k >= 0; --k) {
            for (int32_t s : by_k[k])
                if (s + 1 != fold) t.mono.push_back(s);
            by_k[k].clear();
        }
        const int64_t m = (int64_t)t.mono.size() - first;
        const int nch = (int)((m + CH - 1) / CH);
        if (nch > 1) t.multi = true;
        const int32_t chunk0 = (int32_t)(t.chunk.size() / 4);
        int missing = n;
        std::fill(has.begin(), has.end(), 0);
        for (int c = 0; c < nch; ++c) {
            const int64_t a = first + (int64_t)c * CH;
            const int cnt = (int)std::min<int64_t>(CH, first + m - a);
            t.chunk.push_back((int32_t)a);
            t.chunk.push_back(cnt);
            t.chunk.push_back((int32_t)(t.slice.size() / 2));
            t.chunk.push_back((int32_t)(t.block.size() / 2));
            std::fill(len.begin(), len.end(), 0);
            for (int b = 0; b < cnt; b += 64) {
                const int sc = std::min(64, cnt - b);
                int quads = 0;
                for (int q = 0; q < sc; ++q) {
                    const int32_t s = t.mono[(size_t)(a + b + q)];
                    const int k = (int)(S.mono_start[s + 1] - S.mono_start[s]);
                    quads = std::max(quads, (k + kQuad - 1) / kQuad);
                }
                const size_t w0 = t.words.size();
                if (w0 / kQuad + (size_t)quads * sc > (size_t)INT32_MAX) return "tables too large";
                t.slice.push_back((int32_t)(w0 / kQuad));
                t.slice.push_back(quads);
                t.words.resize(w0 + (size_t)quads * sc * kQuad, pad_word);
                // groups of 16 lanes (one lane per monomial) choose their
                // factors position by position
                for (int g = 0; g < sc; g += 16) {
                    const int lanes = std::min(16, sc - g);
                    int kmax_g = 0;
                    for (int q = 0; q < lanes; ++q) {
                        const int32_t s = t.mono[(size_t)(a + b + g + q)];
                        const int64_t e0 = S.mono_start[s], k = S.mono_start[s + 1] - e0;
                        list.resize((size_t)k);
                        for (int64_t j = 0; j < k; ++j) {
                            const int pos = S.pos[e0 + j];
                            list[(size_t)j] = (uint16_t)((S.exp[e0 + j] - 1) * n + pos);
                            ++len[(size_t)pos];
                        }
                        pool[q].fill(list.data(), (int)k, [](uint16_t v) { return v & 15; });
                        kmax_g = std::max(kmax_g, (int)k);
                    }
                    Pool *lane_pool[16];
                    int bank[16];
                    for (int q = 0; q < lanes; ++q) lane_pool[q] = &pool[q];
                    for (int j = 0; j < kmax_g; ++j) {
                        choose_banks(lane_pool, lanes, bank);
                        for (int q = 0; q < lanes; ++q)
                            if (bank[q] >= 0)
                                t.words[w0 + ((size_t)(j / kQuad) * sc + g + q) * kQuad + j % kQuad] =
                                    pool[q].pop(bank[q]);
                    }
                }
            }
            for (int o = 0; o < n; ++o)
                if (len[(size_t)o] && !has[(size_t)o]) {
                    has[(size_t)o] = 1;
                    --missing;
                }
            // outputs by run length, longest first (stable counting sort)
            const int lmax = cnt;
            bin.assign((size_t)lmax + 2, 0);
            for (int o = 0; o < n; ++o) ++bin[(size_t)(lmax - len[(size_t)o]) + 1];
            for (int l = 0; l <= lmax; ++l) bin[(size_t)l + 1] += bin[(size_t)l];
            for (int o = 0; o < n; ++o) {
                const int j = bin[(size_t)(lmax - len[(size_t)o])]++;
                rank[(size_t)o] = j;
                order[(size_t)j] = o;
            }
            for (int j = 0; j < n_rank; ++j)
                t.out.push_back(j < n ? (uint16_t)order[(size_t)j] : (uint16_t)0xFFFF);
            const size_t blk0 = t.block.size();
            for (int b = 0; b < t.n_blk; ++b) {
                const int rows = (len[(size_t)order[(size_t)b * kRankBlock]] + kParts - 1) / kParts;
                if (rows_total + rows > (int64_t)INT32_MAX / (kRankBlock * kParts))
                    return "tables too large";
                t.block.push_back((int32_t)rows_total);
                t.block.push_back(rows);
                rows_total += rows;
            }
            t.runs.resize((size_t)rows_total * kRankBlock * kParts, (uint16_t)0);
            // the outputs' terms, one output after another, in monomial order
            first_term.assign((size_t)n + 1, 0);
            for (int o = 0; o < n; ++o) first_term[(size_t)o + 1] = first_term[(size_t)o] + len[(size_t)o];
            terms.resize((size_t)first_term[(size_t)n]);
            std::copy(first_term.begin(), first_term.end() - 1, at.begin());
            for (int i = 0; i < cnt; ++i) {
                const int32_t s = t.mono[(size_t)(a + i)];
                for (int64_t e = S.mono_start[s]; e < S.mono_start[s + 1]; ++e)
                    terms[(size_t)at[(size_t)S.pos[e]]++] = (uint16_t)(i | (S.exp[e] << kEntryBits));
            }
            // 16 lanes take eight runs, two terms of each (parts p and p + 2:
            // two lanes per run)
            for (int blk = 0; blk < t.n_blk; ++blk) {
                const size_t row0 = (size_t)t.block[blk0 + 2 * (size_t)blk];
                const int rows = t.block[blk0 + 2 * (size_t)blk + 1];
                for (int h = 0; h < kRankBlock; h += 8) {
                    for (int q = 0; q < 8; ++q) {
                        const int j = blk * kRankBlock + h + q;
                        const int o = j < n ? order[(size_t)j] : -1;
                        pool[q].fill(o < 0 ? nullptr : terms.data() + first_term[(size_t)o],
                                     o < 0 ? 0 : len[(size_t)o], [](uint16_t v) { return v & 15; });
                    }
                    Pool *lane_pool[16];
                    int bank[16];
                    for (int q = 0; q < 16; ++q) lane_pool[q] = &pool[q % 8];
                    for (int r = 0; r < rows; ++r)
                        for (int part = 0; part < 2; ++part) {
                            uint16_t *row = t.runs.data() + ((row0 + (size_t)r) * kRankBlock + (size_t)h) * kParts;
                            choose_banks(lane_pool, 16, bank);
                            for (int q = 0; q < 16; ++q)
                                if (bank[q] >= 0)
                                    row[q % 8 * kParts + part + q / 8 * 2] = pool[q % 8].pop(bank[q]);
                        }
                }
            }
        }
        t.poly.push_back(chunk0);
        t.poly.push_back(chunk0 + nch);
        t.poly.push_back(fold);
        t.poly.push_back(missing == 0);
        t.complete = t.complete || missing == 0;
    }
    t.n_chunks = (int)(t.chunk.size() / 4);
    return std::string();
}

}  // namespace pe
