// Arithmetic of the work split that kernels and host share.  Nothing but constexpr functions of plain values, so that a host
// compiler can run what the kernels run.
#ifndef CF_PLAN_ARITH_H
#define CF_PLAN_ARITH_H

#include <stdint.h>

namespace cf {

constexpr int kMaxRows = 16;               // batch rows of a call at most
constexpr int kMaxKvSplits = 64;           // splits of a batch row's cached tokens at most

// n / d for r = 1 / d to within an ulp or two: n + 1/2 is 0.5 / d away from a multiple, so the quotient is exact for n < 2^20.
// Beyond that it can be one off and more, in either direction.
constexpr int fdiv(int n, float r) { return (int)(((float)n + 0.5f) * r); }

constexpr int larger(int a, int b) { return a > b ? a : b; }
constexpr int smaller(int a, int b) { return a < b ? a : b; }

// ---- Attention items dealt by the lengths of the rows (Params::ragged): row b is cut into splits of about the same number of
// tokens in all rows, at most one item per member, and the items are numbered row by row.
//
// Lengths go up to 2^24, where fdiv is not exact.  What has to hold at every length rests on no quotient: at most `ts` items (a
// size is taken only where the very counts that make the items have been added up) and splits that meet and end with the row.

// Tokens that the longest attention item has to get shorter by for the items to be dealt by the rows' lengths: 48 KB of keys and
// values, what a compute unit streams in 1.5 us; dealing and a merge with splits of their own number cost up to 1 us.  The kernel looks
// for it where a split of the plan is four times that long (finding out takes 0.2 us).  Us a layer, plan / dealt: Llama-3-8B shape, batch
// 4, 5120 to 8192 tokens (1024 against 864 a member) 40.9 / 39.7, 8192 and three of 170 36.1 / 31.4; 16 heads of 64 over 8, batch 6,
// 9000 and five of 190 29.9 / 24.4.  Dealt where it gains less: Llama-3-8B shape, batch 2, 6144 and 8192 (516 against 456) 33.9 / 34.3.
constexpr int ragged_gain(int head_dim) { return 48 * 1024 / (4 * head_dim); }

constexpr int splits_of(int len, int size, float r) { return larger(fdiv(len + size - 1, r), 1); }       // r = 1 / size

// Tokens per split, 0 where the items stay those of the plan (`tps` tokens a split): the fewest of 64 candidates that need at most
// `ts` items, between what a perfect division would take (and 64 splits of a row) and what suffices in whole numbers (an item more
// than it for every row); no fewer than 64, below which a split costs more than it saves.  None may fit: with as many rows as
// members the longest row is the only candidate that can, and the quotient of 2 len - 1 and len may come out as 2.
// Wave: reciprocal(d); len(b), cached tokens of row b; first_of(candidate, fits): the first candidate(k), k < 64, that fits, or 0.
template <class Wave>
constexpr int dealt_size(const Wave &w, int total, int longest, int rows, int ts, int tps, int gain)
{
    auto up = [&](int n, int d) { return fdiv(n + d - 1, w.reciprocal(d)); };
    const int lo = larger(larger(up(total, ts), up(longest, kMaxKvSplits)), 64);
    if (tps - lo < gain) return 0;
    const int hi = ts > rows ? larger(up(total, ts - rows), lo) : larger(longest, lo);
    const int size = w.first_of([&](int k) { return k == 63 ? hi : lo + (int)((float)(hi - lo) * ((float)k * (1.f / 63.f))); },
                                [&](int cand) {
                                    const float r = w.reciprocal(cand);
                                    int need = 0;
                                    for (int b = 0; b < rows; ++b) need += splits_of(w.len(b), cand, r);
                                    return need <= ts;
                                });
    return size > 0 && tps - size >= gain ? size : 0;
}

// Splits of a row of `len` tokens under a dealt size (no more than were counted above).
constexpr int dealt_splits(int len, int size, float r) { return smaller(splits_of(len, size, r), kMaxKvSplits); }

// Tokens [t0, t1) of split `s` of `ns` of a row of `len` tokens; `member` handles it, and member - 1 the split in front of it.
struct TokenRange {
    int t0, t1;
};
template <class Wave>
constexpr TokenRange dealt_range(const Wave &w, int len, int s, int ns, int member, int pairmap)
{
    auto up = [&](int n, int d) { return fdiv(n + d - 1, w.reciprocal(d)); };
    // (the split with the new token is shorter, by about what the token costs)
    int t = up(len + (ns > 1 ? 64 : 0), ns);
    if (t * (ns - 1) > len) t = up(len, ns);
    // (an item of an odd member, on a slower die, is 2 TD shorter than its neighbours: a boundary in front of one is TD further)
    const int td = pairmap && t >= 256 ? 32 : 0;
    return {s == 0 ? 0 : smaller(s * t + (member & 1 ? td : 0), len), s == ns - 1 ? len : smaller(s * t + t + (member & 1 ? 0 : td), len)};
}

}  // namespace cf

#endif
