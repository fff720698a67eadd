// Arithmetic of the work split that kernels and host share.  Nothing but constexpr functions of plain values, so that a host
// compiler can run what the kernels run.
#ifndef CF_PLAN_ARITH_H
#define CF_PLAN_ARITH_H

#include <stddef.h>
#include <stdint.h>

namespace cf {

constexpr int kMaxRows = 16;               // batch rows of a call at most
constexpr int kMaxKvSplits = 64;           // splits of a batch row's cached tokens at most

constexpr size_t kLdsLimit = 160 * 1024 - 256;       // LDS per workgroup on gfx950, minus what a kernel declares statically

// Division by a plan constant d, m = divisor(d) = ceil(2^31 / d): the high half of 2 n m is n / d for n d < 2^31.  Integer division by
// a run-time value costs some thirty instructions.
constexpr uint32_t divisor(int d) { return (uint32_t)((0x80000000ull + d - 1) / d); }
constexpr int qdiv(int n, uint32_t m) { return (int)(((uint64_t)((uint32_t)n + (uint32_t)n) * m) >> 32); }
constexpr int qmod(int n, int d, uint32_t m) { return n - qdiv(n, m) * d; }

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
    // (An item of an odd member, on a slower die, is 2 td shorter than its neighbours: a boundary in front of one is td further.  What it
    // is worth depends on the lengths and is small: us a pass, td 32 / 16 / 0, Llama-3-8B shape, 860 tokens a member 79.1 / 78.6 / 78.6, 280
    // 62.8 / 63.4 / 63.4, 480 67.8 / 68.0 / 68.2, 400 66.5 / 66.3 / 65.9, eight rows, 700 41.7 / 41.4 / 41.1, 1000 59.1 / 59.3 / 59.9; Llama-2-7B
    // shape, 576 83.9 / 83.7 / 84.2; Llama-2-70B shape, 1100 85.0 / 85.1 / 85.3; 32 heads of 64 over 8, 1170 30.4 / 30.1 / 29.9; 8 heads of
    // 128, batch 3, 10667 to 16000 tokens, 82.3 / 78.6 / 81.6.)
    const int td = pairmap && t >= 256 ? 32 : 0;
    return {s == 0 ? 0 : smaller(s * t + (member & 1 ? td : 0), len), s == ns - 1 ? len : smaller(s * t + t + (member & 1 ? 0 : td), len)};
}

// ---- Hidden units of the FFN block's workgroups (vector kernel).  Workgroup w runs on die w % 8, and the odd dies get 3 to 10 % less
// memory bandwidth than the even ones (on every card measured; where they do not, an even share is 2.4 % longer than it need be):
// of the units of two neighbours the even one takes 524 of 1024.  Us a layer, even share 50.0 / 51.2 / 52.4 %: 4096 x 11008 46.2 /
// 45.75 / 46.0, 4096 x 14336 57.1 / 57.0 / 57.5, 8192 x 28672 211.3 / 209.6 / 209.7.
namespace ffn {
constexpr int kThreads = 512;
constexpr int kPiece = 512;                // columns of a row that a wavefront takes in one step
constexpr int kEvenShare = 524;
constexpr int even_units(int pair) { return (pair * kEvenShare + 512) >> 10; }
// first unit of workgroup w of W (even where the shares are uneven)
constexpr int first_unit(int w, int F, int W, int uneven)
{
    if (!uneven) return (int)((long long)w * F / W);
    const int p0 = (int)((long long)(w & ~1) * F / W);
    return w & 1 ? p0 + even_units((int)((long long)(w + 1) * F / W) - p0) : p0;
}
constexpr int most_units(int F, int W, int uneven)       // of a workgroup
{
    const int equal = (F + W - 1) / W;
    return uneven ? larger(even_units((F + W / 2 - 1) / (W / 2)), equal) : equal;
}
// LDS of a batch tile: rows of z, sums of the pieces, g; or the partial output on its way out, 4096 floats
constexpr size_t lds_bytes(int d_model, int batch_tile, int units)
{
    const size_t nck = (d_model + kPiece - 1) / kPiece, dp = nck * kPiece;
    const size_t stages_ab = (size_t)batch_tile * dp / 2 + 2 * (size_t)batch_tile * units * nck + (size_t)batch_tile * units;
    return (stages_ab > (size_t)(8 * kThreads) ? stages_ab : (size_t)(8 * kThreads)) * sizeof(float);
}
// Uneven shares where workgroups come in whole rounds of the dies and the larger share still fits LDS at the largest batch tile.
constexpr int uneven_shares(int d_model, int F, int W, int largest_tile)
{
    return W % 8 == 0 && lds_bytes(d_model, largest_tile, most_units(F, W, 1)) <= kLdsLimit;
}
}  // namespace ffn

}  // namespace cf

#endif
