// The split arithmetic of cf_plan_arith.h as the host compiler sees it, for tests.  What the kernel does with the lanes of a
// wavefront is a loop here; reciprocals are off by a given number of ulps, since the device's may be.
#include "../../paper_2508_18850_amd/csrc/cf_plan_arith.h"

#include <cmath>

namespace {
float reciprocal(int d, int ulps)
{
    float r = 1.0f / (float)d;
    for (int i = 0; i < (ulps < 0 ? -ulps : ulps); ++i) r = std::nextafter(r, ulps > 0 ? 2.0f : 0.0f);
    return r;
}
struct HostWave {
    const int *lens;
    int ulps;
    float reciprocal(int d) const { return ::reciprocal(d, ulps); }
    int len(int b) const { return lens[b]; }
    template <class Candidate, class Fits>
    int first_of(Candidate &&candidate, Fits &&fits) const
    {
        for (int k = 0; k < 64; ++k)
            if (fits(candidate(k))) return candidate(k);
        return 0;
    }
};
}  // namespace

extern "C" {

int pa_ragged_gain(int head_dim) { return cf::ragged_gain(head_dim); }

// The first n of `count` values whose quotient by d is not the integer one, or -1.
int pa_qdiv_differs(const int *n, int count, int d)
{
    for (int i = 0; i < count; ++i)
        if (cf::qdiv(n[i], cf::divisor(d)) != n[i] / d || cf::qmod(n[i], d, cf::divisor(d)) != n[i] % d) return n[i];
    return -1;
}
int pa_fdiv_differs(const int *n, int count, int d, int ulps)
{
    for (int i = 0; i < count; ++i)
        if (cf::fdiv(n[i], reciprocal(d, ulps)) != n[i] / d) return n[i];
    return -1;
}

int pa_first_unit(int w, int F, int W, int uneven) { return cf::ffn::first_unit(w, F, W, uneven); }
int pa_most_units(int F, int W, int uneven) { return cf::ffn::most_units(F, W, uneven); }
int pa_uneven_shares(int d_model, int F, int W, int tile) { return cf::ffn::uneven_shares(d_model, F, W, tile); }
int pa_lds_bytes(int d_model, int tile, int units) { return (int)cf::ffn::lds_bytes(d_model, tile, units); }
int pa_lds_limit() { return (int)cf::kLdsLimit; }

// Deals `rows` rows of the given lengths.  Returns the number of items (0: the plan's); `splits`: per row; `range`: t0, t1 of every
// item in order (room for 16 * 64).
int pa_deal(int rows, const int *lens, int ts, int tps, int gain, int pairmap, int ulps, int *size_out, int *splits, int *range)
{
    const HostWave w = {lens, ulps};
    int total = 0, longest = 0;
    for (int b = 0; b < rows; ++b) {
        total += lens[b];
        longest = lens[b] > longest ? lens[b] : longest;
    }
    const int size = cf::dealt_size(w, total, longest, rows, ts, tps, gain);
    *size_out = size;
    if (size == 0) return 0;
    int items = 0;
    for (int b = 0; b < rows; ++b) {
        splits[b] = cf::dealt_splits(lens[b], size, w.reciprocal(size));
        for (int s = 0; s < splits[b]; ++s, ++items) {
            const cf::TokenRange r = cf::dealt_range(w, lens[b], s, splits[b], items, pairmap);
            range[2 * items] = r.t0, range[2 * items + 1] = r.t1;
        }
    }
    return items;
}

}  // extern "C"
