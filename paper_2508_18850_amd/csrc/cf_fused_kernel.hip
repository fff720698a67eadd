// Fused decode-block kernel for gfx950: QKV projection + RoPE + KV append +
// split-KV attention + output projection in one launch (paper Alg. 3).
//
// Mapping.  The paper maps one attention head to a cluster of thread blocks and
// resolves the dependencies between the blocks of a cluster with ClusterGather
// and ClusterReduce over distributed shared memory.  gfx950 has no clusters, so
// a "team" of workgroups (with an even number of members and 4 | n_kv_heads on
// one pair of XCDs) serves one KV head
// together with the query heads that use it.  Every member streams, in this
// order, so that each dependency falls behind a stream that does not need it:
//   1a  its slice of the reduction dimension of the team's W_q columns
//       (split-K instead of the paper's split of the head dimension: rows of 256
//       contiguous bytes coalesce, 32 columns would not)
//   1b  the same slice of the team's W_k / W_v columns
//   2   the first K/V rows are put in flight, then the q partials of the team
//       are summed (the role of ClusterGather) and rotated; online-softmax
//       attention over the member's slice of the cached sequence (Alg. 3 step
//       4); the member with the last slice also sums the k/v partials, appends
//       the new key/value and counts the new token
//   3   its block of W_o is loaded into registers, then the split-KV partials of
//       the head are merged (Alg. 3 steps 5-7, local sums rescaled by
//       exp(m_i - M) before being added) and multiplied (step 8) into a per-head
//       partial of the output
//   4   every workgroup adds, over all heads and in a fixed order, the partials
//       of its own few output columns (the paper uses atomicAdd) and writes fp16.
// Exchange between workgroups needs no counters: every exchanged fp32 value is
// stored as a 64-bit {value, stamp} pair with one write-through store, the stamp
// being the launch number; a reader polls the pair until the stamp is current.
// Every workgroup counts the launches it has completed; the count gives the launch number.  All
// workgroups of the launch must be resident (checked on the host), since
// readers spin.  Spins are bounded: after spin_ticks a thread sets an error
// flag and goes on, so the kernel always ends.
#include "cf_lanes_device.h"
#include "cf_mfma_device.h"
#include "cf_params.h"
#include "cf_rope_device.h"
#include "cf_stream_device.h"

#include <cstddef>
#include <type_traits>

namespace cf {
namespace {

// CF_LAYER=1 compiles the kernel with the RMSNorm prologue, the residual epilogue and per-row positions
// (fused_decode_layer); without it none of that code is in the kernel (fused_decode_block).
#ifndef CF_LAYER
#define CF_LAYER 0
#endif
#if CF_LAYER
#define CF_KERNEL fused_decode_layer
#else
#define CF_KERNEL fused_decode_block
#endif
constexpr bool kLayer = CF_LAYER != 0;
constexpr int NT = kThreads;
constexpr int NW = kWaves;
constexpr float kNegBig = -1.0e30f;   // stands for "no score yet"; finite so that differences never give NaN
#ifndef CF_PREFETCH_NEXT_LAYER
#define CF_PREFETCH_NEXT_LAYER 1
#endif
constexpr bool kPrefetchNextLayer = CF_PREFETCH_NEXT_LAYER != 0;   // stack kernel: next layer's first weights during the tail

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

using Stream = Part<2>;

__device__ __forceinline__ void unpack8(const h8 &u, float (&f)[8])
{
#pragma unroll
    for (int k = 0; k < 8; ++k) f[k] = (float)u[k];
}

// Batch tile 16: the two projections (Alg. 3 steps 2 and 8) are dense [16 x K] x [K x N]
// products and run on MFMA tiles (v_mfma_f32_16x16x32_f16: A is 16 x 32, B is 32 x 16, fp32 accumulators).
// Operand layout of that instruction: lane l holds, of A, row l % 16 and eight consecutive values of the
// contraction index for group l / 16; of B, column l % 16 and the same eight contraction values; of the
// result, column l % 16 and rows 4 * (l / 16) + 0..3.  The weights stay in the layout the batch-1 path
// streams (a lane loads eight COLUMNS of one row), so eight loaded rows are transposed inside the lane
// into eight operands of one column each (transpose8); the sixteen batch rows are the A operand.
template <int HD, int BT>
struct Mfma {
    static constexpr bool on = mfma_tiles(BT);
};
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 mfma16(const h8 &a, const h8 &b, const f32x4 &c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// w[u] = row u, eight adjacent columns  ->  f[c] = column c, rows 0..7 (a 8 x 8 transpose of 16-bit values
// inside one lane: one byte permute per result register)
__device__ __forceinline__ void transpose8(const h8 *w, h8 (&f)[8])
{
#pragma unroll
    for (int c2 = 0; c2 < 4; ++c2) {
        u32x4 e, o;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const uint32_t lo = __builtin_bit_cast(u32x4, w[2 * d])[c2], hi = __builtin_bit_cast(u32x4, w[2 * d + 1])[c2];
            e[d] = __builtin_amdgcn_perm(hi, lo, 0x05040100u);    // {lo.low half, hi.low half}
            o[d] = __builtin_amdgcn_perm(hi, lo, 0x07060302u);    // {lo.high half, hi.high half}
        }
        f[2 * c2] = __builtin_bit_cast(h8, e);
        f[2 * c2 + 1] = __builtin_bit_cast(h8, o);
    }
}

// v = hi + lo with both parts fp16, for operands that enter a sum of exponents or weights of at most one: 22 bits of values
// around one, an absolute step of 2^-24 below, no more than 65504.  Operands of the projections: mfma::split_scaled.
__device__ __forceinline__ void split_hi_lo(const float (&v)[8], h8 &hi, h8 &lo)
{
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        hi[k] = (_Float16)v[k];
        lo[k] = (_Float16)(v[k] - (float)hi[k]);
    }
}

__device__ __forceinline__ float h2f(uint16_t bits) { return (float)__builtin_bit_cast(_Float16, bits); }
__device__ __forceinline__ uint16_t f2h(float v) { return __builtin_bit_cast(uint16_t, (_Float16)v); }

using lanes::dpp_move;

// Sum over the LPR (8 or 16) consecutive lanes that hold one row; every lane gets the total.
template <int LPR>
__device__ __forceinline__ float row_sum(float v)
{
    v += dpp_move<0xB1>(v);    // quad_perm [1,0,3,2]
    v += dpp_move<0x4E>(v);    // quad_perm [2,3,0,1]
    v += dpp_move<0x141>(v);   // row_half_mirror: lane i <-> 7-i within 8 lanes
    if (LPR == 16) v += dpp_move<0x140>(v);   // row_mirror: lane i <-> 15-i within 16 lanes
    return v;
}

// Workgroup barrier that orders LDS accesses only.  __syncthreads() would also wait for every
// outstanding global load of the wave (vmcnt(0)), which would drain the loads that are kept in
// flight across phases; nothing here passes data between the threads of a workgroup through
// global memory.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ float wave_sum(float v)
{
    return lanes::sum_groups<16>(row_sum<16>(v));
}

// Maximum / sum over the wavefront, the same value in every lane: four data-parallel-primitive steps inside each row of
// 16 lanes, then the four row results are read out as scalars (no trip through the LDS crossbar).
__device__ __forceinline__ float lane_of(float v, int l) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l)); }
__device__ __forceinline__ float wave_max(float v)
{
    v = fmaxf(v, dpp_move<0xB1>(v));
    v = fmaxf(v, dpp_move<0x4E>(v));
    v = fmaxf(v, dpp_move<0x141>(v));
    v = fmaxf(v, dpp_move<0x140>(v));
    return fmaxf(fmaxf(lane_of(v, 0), lane_of(v, 16)), fmaxf(lane_of(v, 32), lane_of(v, 48)));
}
// The bits of the largest magnitude over the wavefront, as a scalar, of up to four values per lane: the four are folded
// into one register first (a row of 16 lanes each), so that they share the steps between lanes.
template <int N>
__device__ __forceinline__ void wave_max_bits(const float (&v)[N], int (&out)[N])
{
    static_assert(N == 1 || N == 2 || N == 4, "folds by halves");
    float h[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        float p = v[2 * j % N], q = v[(2 * j + 1) % N];
        lanes::swap32(p, q);
        h[j] = fmaxf(fabsf(p), fabsf(q));            // lanes 0..31: value 2 j, lanes 32..63: value 2 j + 1
    }
    lanes::swap16(h[0], h[1]);
    const int m = __builtin_bit_cast(int, lanes::max_row(fmaxf(h[0], h[1])));        // rows of lanes: values 0, 2, 1, 3
#pragma unroll
    for (int n = 0; n < N; ++n) out[n] = __builtin_amdgcn_readlane(m, 32 * (n & 1) + 16 * (n >> 1));
}
__device__ __forceinline__ float wave_total(float v)
{
    v = row_sum<16>(v);
    return (lane_of(v, 0) + lane_of(v, 16)) + (lane_of(v, 32) + lane_of(v, 48));
}

// Exchange slots (partials handed from one workgroup to another).  A slot is a 64-bit
// {fp32 bits, stamp} pair written by ONE 8-byte write-through store (agent scope), so a
// reader sees either the old pair or the new one; the stamp of a launch is its number.  Indices are 32 bits (the host checks that
// an area is smaller than 4 GiB).
//
// Scope: agent (sc1, through to memory), also for slots that only travel inside a team.  Keeping
// those in the L2 of the team's die (workgroup-scope loads and stores) was tried: the per-CU cache
// then serves the polled line and the reader never sees the new stamp.
struct Xbuf {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ explicit Xbuf(const void *base)
        : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, 0xfffffff8u, 0x00020000)) {}
    __device__ __forceinline__ u32x2 ld(uint32_t idx) const
    {
        return __builtin_amdgcn_raw_buffer_load_b64(r, idx * 8, 0, 16);
    }
    // two neighbouring pairs (idx even): each half carries its own stamp, so nothing rests on the 16 bytes arriving together
    __device__ __forceinline__ u32x4 ld2(uint32_t idx) const
    {
        return __builtin_amdgcn_raw_buffer_load_b128(r, idx * 8, 0, 16);
    }
    __device__ __forceinline__ void st(uint32_t idx, float v, uint32_t stamp) const
    {
        u32x2 d = {__builtin_bit_cast(uint32_t, v), stamp};
        __builtin_amdgcn_raw_buffer_store_b64(d, r, idx * 8, 0, 16);
    }
};

// Bounded spinning: returns true when the caller should give up.
struct Spin {
    long long t0 = 0;
    __device__ __forceinline__ bool expired(const Params &p)
    {
        __builtin_amdgcn_s_sleep(1);
        const long long now = wall_clock64();
        if (t0 == 0) t0 = now;
        if (now - t0 >= (long long)p.spin_ticks) {            // a limit of 0 gives up at the first failed look
            __hip_atomic_store(p.err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return true;
        }
        return false;
    }
};

// Sum of n stamped slots base, base+stride, ... in index order; spins until all are current.
// Loads go out eight at a time (indices past n repeat the last slot and are ignored) and are consumed
// only after all eight have been issued: written as one loop, each load was waited for on its own.
template <int C = 8>
__device__ __forceinline__ float ll_sum(const Params &p, const Xbuf &x, uint32_t base, uint32_t stride, int n,
                                        uint32_t stamp)
{
    Spin spin;
    for (;;) {
        float s = 0.f;
        uint32_t stale = 0;                   // bits in which a stamp differs from the current one
        if (n == 1) {
            const u32x2 v = x.ld(base);
            stale = v.y ^ stamp;
            s = __builtin_bit_cast(float, v.x);
        } else {
            for (int k0 = 0; k0 < n; k0 += C) {
                u32x2 v[C];
#pragma unroll
                for (int k = 0; k < C; ++k) v[k] = x.ld(base + (uint32_t)min(k0 + k, n - 1) * stride);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int k = 0; k < C; ++k) {
                    stale |= v[k].y ^ stamp;
                    s += k0 + k < n ? __builtin_bit_cast(float, v[k].x) : 0.f;
                }
            }
        }
        if (stale == 0 || spin.expired(p)) return s;
    }
}

// First weight column of selector `sel` for a team: sel < G query heads, G = key, G+1 = value.
// Tokens cached for batch row b == index of the row's new token (b is uniform over the workgroup).
// Values outside 0 .. pos are clamped, so that a bad entry cannot make the kernel leave its buffers.
__device__ __forceinline__ int row_pos(const Params &p, int b)
{
    if (kLayer && p.row_pos) return min(max(__builtin_amdgcn_readfirstlane(p.row_pos[b]), 0), p.pos);
    return p.pos;
}

// The attention item of a member where the batch rows have lengths of their own (Params::ragged).
struct RowItem {
    int b = 0, s = 0, ns = 1, pos = 0;      // row, split, splits of the row, its cached tokens
    int first = 0;                          // number of the row's first item
    int t0 = 0, t1 = 0;
    int table = 0;                          // lane b: first item of row b (lanes past the batch: number of items)
    int items = 0;                          // 0: the plan's items
};
// The lanes of a wavefront as dealt_size wants them: the length of row `lane % 16` and one candidate each.
struct DealWave {
    int lane, own;
    __device__ __forceinline__ float reciprocal(int d) const { return cf::reciprocal(d); }
    __device__ __forceinline__ int len(int b) const { return __builtin_amdgcn_readlane(own, b); }
    template <class Candidate, class Fits>
    __device__ __forceinline__ int first_of(Candidate &&candidate, Fits &&fits) const
    {
        const int c = candidate(lane);
        const unsigned long long m = __ballot(fits(c));
        return m ? __builtin_amdgcn_readlane(c, __builtin_ctzll(m)) : 0;
    }
};
// `len`: cached tokens of row `lane % 16` (0 past the batch).  All wavefronts of all workgroups come to the same result.
template <int CTRL>
__device__ __forceinline__ int dpp_int(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true); }
template <int HD>
__device__ __forceinline__ RowItem deal_rows(const Params &p, int lane, int len, int member, RowItem it)         // it: the plan's item
{
    int total = len, longest = len;                               // over the 16 lanes of a row
    total += dpp_int<0xB1>(total), longest = max(longest, dpp_int<0xB1>(longest));       // quad_perm [1,0,3,2]
    total += dpp_int<0x4E>(total), longest = max(longest, dpp_int<0x4E>(longest));       // quad_perm [2,3,0,1]
    total += dpp_int<0x141>(total), longest = max(longest, dpp_int<0x141>(longest));     // row_half_mirror
    total += dpp_int<0x140>(total), longest = max(longest, dpp_int<0x140>(longest));     // row_mirror
    total = __builtin_amdgcn_readfirstlane(total), longest = __builtin_amdgcn_readfirstlane(longest);
    const DealWave wave = {lane, len};
    const int size = dealt_size(wave, total, longest, p.B, p.TS, p.TPS, ragged_gain(HD));
    if (size == 0) return it;
    const int row = lane & 15;
    const int mine = row < p.B ? dealt_splits(len, size, reciprocal(size)) : 0;          // splits of the lane's row
    int incl = mine;                                              // ... and of those before it
    incl += dpp_int<0x111>(incl);                                 // row_shr 1, 2, 4, 8
    incl += dpp_int<0x112>(incl);
    incl += dpp_int<0x114>(incl);
    incl += dpp_int<0x118>(incl);
    it.items = __builtin_amdgcn_readlane(incl, 15);
    it.table = lane < 16 ? incl - mine : it.items;
    it.b = max(__builtin_popcountll(__ballot(lane < p.B && it.table <= member)) - 1, 0);
    it.first = __builtin_amdgcn_readlane(it.table, it.b);
    it.ns = __builtin_amdgcn_readlane(mine, it.b);
    it.pos = __builtin_amdgcn_readlane(len, it.b);
    it.s = member - it.first;
    if (member < it.items) {
        const TokenRange r = dealt_range(wave, it.pos, it.s, it.ns, member, p.pairmap);
        it.t0 = r.t0, it.t1 = r.t1;
    }
    return it;
}

template <int G>
__device__ __forceinline__ int qkv_block(const Params &p, int team, int sel)        // in blocks of head_dim columns
{
    return sel < G ? team * G + sel : p.nq + team + (sel - G) * p.nkv;
}
template <int HD, int G>
__device__ __forceinline__ int qkv_col0(const Params &p, int team, int sel) { return qkv_block<G>(p, team, sel) * HD; }

// The RoPE tables in LDS: [rows][HD] floats, per row HD/2 cosines then HD/2 sines of that row's position.
// One row (the common position) unless the rows of the batch have positions of their own.
template <int HD, int BT>
struct RopeRows {
    static constexpr int ROWS = kLayer ? BT : 1;                      // rows the LDS array has room for
    static constexpr int NE = (ROWS * (HD / 2) + NT - 1) / NT;        // table entries per thread
};

// ---------------------------------------------------------------------------
// Phase 1 (Alg. 3 step 2, split over the reduction dimension).  The member owns the
// row slice ks of W_qkv and, within it, the column blocks ("selectors") sel0, sel0+dsel,
// ... of the team: query heads first, then key / value.  All (selector, row batch)
// steps run as one software pipeline: the loads of step k+1 are issued before step k is
// consumed, also across selectors and across the partial-sum epilogues, and the loads
// of the NEXT phase (issue_next) are issued before the last step is consumed, so the
// memory pipe never drains.
// ---------------------------------------------------------------------------
// Per-phase time stamps (cf_debug_export what = 2) are compiled in only with -DCF_STAMPS=1: their
// `if (thread 0)` blocks cost a quarter of a microsecond per step.  A stamp goes to LDS and is copied to
// memory when the workgroup ends: a store to memory in the first microseconds of a kernel (the first
// version did that) holds up every load behind it for about 3 us and falsifies what it measures.
#ifndef CF_STAMPS
#define CF_STAMPS 0
#endif
#if CF_STAMPS
__shared__ unsigned long long s_ts[kStamps];
#define CF_STAMP(k)                                       \
    do {                                                  \
        if (threadIdx.x == 0) s_ts[k] = wall_clock64();   \
    } while (0)
#else
#define CF_STAMP(k)
#endif

// The launch stamp of layer `layer` of a launch whose first layer has count cnt0 (never 0, the value of a
// cleared slot: the low word plus the number of times it has wrapped).
__device__ __forceinline__ uint32_t stamp_of(unsigned long long cnt0, int layer)
{
    const unsigned long long cnt = cnt0 + (unsigned long long)layer;
    return (uint32_t)(cnt + (cnt >> 32));
}

// The two batches of weight rows that phase 1 keeps in flight, and the cursor of the next batch to load.  They live
// outside p1_all so that, in a stack of layers, the first two batches of the NEXT layer can be requested while the
// current layer still exchanges its last partial results (its memory pipe would idle otherwise).
template <int HD, int BT>
struct P1Cfg {
    static constexpr bool MF = Mfma<HD, BT>::on;
    static_assert(MF || BT <= 4, "vector tiles of up to four rows");
    static constexpr int U = BT == 4 ? 4 : 8;                               // loads per thread and batch
};
// How many of the two batches a stack requests ahead for its next layer: what the registers of the variant allow
// (none with the 16-row tile, one where the attention or a second query head per KV head takes the room).
template <int HD, int G, int BT>
struct P1Ahead {
    static constexpr int n = !kPrefetchNextLayer || BT > 4 ? 0 : (G >= 2 && BT == 1 ? 1 : 2);
};
template <int HD, int BT>
struct P1Regs {
    h8 wa[P1Cfg<HD, BT>::U], wb[P1Cfg<HD, BT>::U];
    int si = 0, i0 = 0;
    uint32_t sbase = 0;
};

// `layer` > 0 (a stack of layers in one launch): the input rows are what the final reduction of the previous layer
// left in the slots xin (stamped fp32 values that are exact fp16 numbers), and cnt0 is known already.
// PART 0: the whole phase (`primed`: its first two batches are in flight already, requested by PART 1 and 2);
// PART 1 / 2: only request the first / second batch of this layer's weights into rg and return.
template <int HD, int G, int BT, bool STACK, int PART, class NextFn>
__device__ __forceinline__ uint32_t p1_all(const Params &p, const LayerPtrs &lp, int tid0, int team, int member, float *smem,
                                           float *rope, int layer, const uint64_t *xin, int n_layers,
                                           unsigned long long &cnt0, P1Regs<HD, BT> &rg, bool primed, int &lens, NextFn &&issue_next)
{
    constexpr int LPR = HD / 8;
    constexpr int NG = NT / LPR;
    // loads per thread and batch: the 4-row tile is best with 4 (8B shape, batch 4: 55.1 us with 8, 53.6 with 4, 53.7 with 2).
    // With MFMA tiles (MF) a batch is eight rows per lane: one step of the contraction, 32 RS rows, per wavefront.
    constexpr bool MF = P1Cfg<HD, BT>::MF;
    constexpr int U = P1Cfg<HD, BT>::U;
    constexpr int MAXI = BT == 1 ? 4 : (BT <= 4 ? 2 : 1);   // selectors whose wave partials are buffered in LDS
    const int tid = tid0, wv = tid >> 6, lig = tid % LPR, grp = tid / LPR;
    const int kg = (tid & 63) >> 4;                         // MF: contraction group of the lane (rows 8 kg .. 8 kg + 7 of a step)
    // MF: the sixteen columns of an operand are LPR 16-byte pieces x RS sets of 32 rows (two sets at head_dim 64)
    constexpr int RS = MF ? 16 / LPR : 1;
    const int rs = tid / LPR % RS;
    const int lrow = 32 * (RS * wv + rs) + 8 * kg;          // MF: first row of the lane inside a batch of 256 RS rows
    const int ks = qmod(member, p.KS, p.div_ks);
    const int sel0 = qdiv(member, p.div_ks), dsel = p.DSEL;
    const int r0 = ks * p.RPS;
    const int nrows = min(p.RPS, p.D - r0);                 // > 0: the host never plans an empty slice
    const int iters = (nrows + NG - 1) / NG;
    const int nb = (iters + U - 1) / U;                     // load batches per selector
    // selectors sel0, sel0 + dsel, ... of the team's G + 2 (the members past KS * DSEL have none)
    const int nsel = sel0 < min(dsel, G + 2) ? qdiv(G + 2 - sel0 + dsel - 1, p.div_dsel) : 0;
    const int nsteps = nsel * nb;
    auto sel_of = [&](int si) { return sel0 + si * dsel; };
    float *xs = smem;                       // [BT][RPS]
    // MF: x as fp16 MFMA operands, [16][XS] halves (rows of an odd number of 16-byte pieces: the sixteen lanes of an operand
    // read then fall into different banks), followed by a second array with the low parts of x * gamma (RMSNorm)
    const int XS = xs16_stride(p.RPS);
    _Float16 *xh = reinterpret_cast<_Float16 *>(smem), *xl = xh + 16 * XS;
    float *red = smem + (MF ? (kLayer || HD == 128 ? 16 : 8) * XS : BT * p.RPS);   // [MAXI][NW][BT][HD]
    const Xbuf x1(p.p1);
    // A selector is a block of head_dim columns, its rows p.wrow bytes apart (row-major: of a whole row; packed: of one
    // contiguous block).  The buffer of a selector begins at the slice's first row and ends behind the block's part of its last.
    const uint32_t rowb = p.wrow, lim = (uint32_t)(nrows - 1) * rowb + HD * 2;
    const uint32_t voff0 = (uint32_t)(MF ? lrow : grp) * rowb + lig * 16;

    // A step is (selector, batch of U row groups).  Steps are loaded and consumed strictly in order,
    // so each side keeps a cursor that is advanced incrementally: no divisions.
    const uint32_t step_b = (uint32_t)NG * rowb;            // bytes between consecutive row groups
    struct Cursor {
        int si, i0;          // selector index, first row group of the batch
        uint32_t sbase;      // offset of that row group's first row
    };
    auto advance = [&](Cursor &c) {
        const bool next = c.i0 + U >= iters;
        c.sbase = next ? 0u : c.sbase + (uint32_t)U * step_b;
        c.i0 = next ? 0 : c.i0 + U;
        c.si += next;
    };
    Cursor cc = {0, 0, 0u};                                 // next step to consume
    Cursor lc = cc;                                         // next step to load
    constexpr int AHEAD = STACK ? P1Ahead<HD, G, BT>::n : 0;
    if (PART == 2 || (PART == 0 && primed && AHEAD > 0)) lc = Cursor{rg.si, rg.i0, rg.sbase};
    // Every call issues exactly U load instructions on one straight-line path, also for a step past
    // the end (an empty buffer).  The compiler derives each wait from
    // the number of loads issued after the one it needs, taking the smallest over all paths of the
    // control flow, so a branch around loads would make every later wait drain the queue.
    auto load = [&](h8(&w)[U], uint32_t voff) {
        const char *base = reinterpret_cast<const char *>(lp.wqkv) + (size_t)r0 * rowb +
                           (size_t)(uint32_t)qkv_block<G>(p, team, sel_of(lc.si)) * p.wblk;
        const Stream W(base, lc.si < nsel ? lim : 0u);
        uint32_t off = voff + lc.sbase;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            w[u] = W.ld(off);
            off += MF ? rowb : step_b;
        }
        advance(lc);
    };

    CF_STAMP(20);           // phase 1 set up
    // Kernel start: the first batch of weights goes out at once, then the small loads (this slice of
    // x, the RoPE frequencies), then the second batch.  Loads return in order: x arrives right behind
    // the first batch and is staged into LDS while the second one streams.
    h8(&wa)[U] = rg.wa;
    h8(&wb)[U] = rg.wb;
    if (PART != 0) {
        // (`primed` here means "there is a next layer"; without one the loads go out past the end of their buffer: the
        // registers are written either way, so that what they held does not stay alive through the caller's loop)
        load(PART == 1 ? wa : wb, primed ? voff0 : kNoLoad);
        rg.si = lc.si;
        rg.i0 = lc.i0;
        rg.sbase = lc.sbase;
        return 0u;
    }
    // (a stack past its first layer has both batches in flight: the branch costs the other path, the first layer
    // of a stack, some exactness of its waits, nothing else)
    if (!(AHEAD >= 1 && primed)) load(wa, voff0);
    __builtin_amdgcn_sched_barrier(0);
    CF_STAMP(12);           // first weight batch issued
    // Outside a stack x goes from memory to LDS in 16-byte pieces, XP of them per thread requested here (value by value it
    // was up to seventeen 2-byte loads per thread, and as many of gamma, in front of the second weight batch, and a
    // round trip per value for slices of more than 1024 rows).  The host makes the slices multiples of eight rows
    // wherever that leaves no slice empty; the others are staged value by value.
    constexpr bool XV = !STACK;
    constexpr bool ROW = STACK && kLayer;                         // the whole row is fetched (below)
    static_assert(!ROW || BT == 1, "one row per launch");
    constexpr int XP = MF && !STACK ? 4 : 2;
    // MFMA tiles of the layer kernel: a row's pieces belong to one half wavefront (up to eight rows: one wavefront), since
    // x * gamma is scaled by the largest value of the row's slice (stage_piece below), and the maximum is then one between lanes.
    constexpr bool BYROW = MF && kLayer && !STACK;
    const int lpr = p.B > 8 ? 32 : 64, brow = p.B > 8 ? tid >> 5 : wv, lane0 = tid & (lpr - 1);
    const bool xvec = STACK || (p.RPS & 7) == 0;          // (the host launches no stack otherwise)
    const int P8 = p.RPS >> 3, npc = xvec ? p.B * P8 : 0;         // pieces of a row's slice, of all rows
    const uint4 *xg4 = reinterpret_cast<const uint4 *>(p.x), *gg4 = reinterpret_cast<const uint4 *>(lp.gamma ? lp.gamma : p.x);
    uint4 xp[XV ? XP : 1], gp[XV ? XP : 1];
    auto piece_of = [&](int i, int &b, int &c) {                  // false: past the rows or past the slice
        b = BT == 1 ? 0 : qdiv(i, p.div_p8);
        c = i - b * P8;
        return i < npc && 8 * c < nrows;
    };
    auto own_piece = [&](int q, int &b, int &c) {                 // piece q of this thread
        if constexpr (!BYROW) return piece_of(tid + q * NT, b, c);
        b = brow;
        c = lane0 + q * lpr;
        return xvec && b < p.B && 8 * c < nrows;
    };
    // The input of a stack comes from stamped slots, two fp16 values and the stamp in eight bytes; in its first layer from x.
    // Without norm and residual a workgroup fetches its slice, in pieces like those above (two 16-byte loads each), XP per
    // thread and round trip, the batch's own rows only; the first trip is requested here.  With norm (batch 1, d_model at most
    // 8 NT) it fetches the whole row, a piece per thread, since it needs its mean square, and stages the pieces of its slice from it.
    const int xn = p.B * p.RPS;
    const float inv_rps = __builtin_amdgcn_rcpf((float)p.RPS);
    auto x_at = [&](int i, int &b, int &r) {                      // value i: row b of the batch, row r of the slice
        b = BT == 1 ? 0 : (int)(((float)i + 0.5f) * inv_rps);     // (exact: i < 2^18, the quotient is 0.5 / RPS away from an integer)
        r = i - b * p.RPS;
        return i < xn && r < nrows;
    };
    const bool from_slots = STACK && layer > 0;
    const Xbuf xsl(xin ? (const void *)xin : (const void *)p.p1);
    u32x4 sp[STACK ? XP : 1][2];                                  // pieces of the slice: {two values, stamp} x 4
    auto piece_slots = [&](int i0) {
        int i = i0 + tid;
        asm volatile("" : "+v"(i));
#pragma unroll
        for (int q = 0; q < XP; ++q) {
            int b, c;
            const size_t at = piece_of(i + q * NT, b, c) ? ((size_t)b * p.D + r0) / 2 + 4 * c : 0;
            sp[q][0] = xsl.ld2(at);
            sp[q][1] = xsl.ld2(at + 2);
        }
    };
    auto piece_values = [&](int i0) {
        int i = i0 + tid;
        asm volatile("" : "+v"(i));
#pragma unroll
        for (int q = 0; q < XP; ++q) {
            int b, c;
            const uint4 v = xg4[piece_of(i + q * NT, b, c) ? ((size_t)b * p.D + r0) / 8 + c : 0];
            sp[q][0] = u32x4{v.x, 0u, v.y, 0u};
            sp[q][1] = u32x4{v.z, 0u, v.w, 0u};
        }
    };
    if constexpr (XV) {
#pragma unroll
        for (int q = 0; q < XP; ++q) {
            int b, c;
            const bool in = own_piece(q, b, c);
            xp[q] = xg4[in ? ((size_t)b * p.D + r0) / 8 + c : 0];
        }
    } else if constexpr (!ROW) {
        if (from_slots)
            piece_slots(0);
        else
            piece_values(0);
    }
    // RMSNorm in front of the projection (when a weight vector is given): the projection is linear, so the
    // weights gamma go into the staged slice of x and the factor 1/sqrt(mean(x^2) + eps) of a row goes into
    // the partial sums when they are stored.  Every workgroup takes the mean square from the whole row
    // (D*2 bytes: one or two 16-byte loads per thread, issued here with the other small loads).
    const bool norm = kLayer && lp.gamma != nullptr;
    if (XV && norm) {       // (a wait behind this branch counts the loads of the path without it: nothing drains)
#pragma unroll
        for (int q = 0; q < XP; ++q) {
            int b, c;
            const bool in = own_piece(q, b, c);
            gp[q] = gg4[in ? r0 / 8 + c : 0];
        }
    }
    float *nrm = red + MAXI * NW * BT * HD;                       // [NW][BT] sums of squares, one per wavefront and row
    constexpr int RG = BT < 4 ? BT : (MF ? 8 : 4);                // rows whose loads are in flight together
    const int d8 = p.D >> 3;                                      // 16-byte pieces of a row
    // Pieces of a row per thread and round: a row has up to 16 NT values; on the 16-row tile the second half of longer rows takes a
    // round of its own.  The loads are in no branch (a buffer that ends with the batch: rows past it and lanes past the row give zeros):
    // behind branches their registers were copied where the paths met, which waited for the first weight batch (Llama-3-8B
    // shape, 4 rows: x staged 1.5 us later).
    constexpr int KR = MF || ROW ? 1 : 2;
    const __amdgpu_buffer_rsrc_t xrows = buffer_of(p.x, norm || ROW ? (uint32_t)(p.B * p.D) * 2 : 0u);
    uint4 xq[RG][KR];                                             // rows b0 .. b0 + RG - 1
    auto load_rows = [&](int b0, int k0) {
#pragma unroll
        for (int r = 0; r < RG; ++r)
#pragma unroll
            for (int k = 0; k < KR; ++k) {
                const int c = tid + (k0 + k) * NT;
                xq[r][k] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                                         xrows, (c < d8 ? (uint32_t)c * 16 : kNoLoad) + (uint32_t)(b0 + r) * p.D * 2, 0, 0));
            }
    };
    auto square_rows = [&](int b0, int k0) {
#pragma unroll
        for (int r = 0; r < RG; ++r) {
            if (b0 + r >= p.B) break;                             // (uniform)
            float ss = 0.f;
#pragma unroll
            for (int k = 0; k < KR; ++k) {
                float f[8];
                unpack8(__builtin_bit_cast(h8, xq[r][k]), f);
                float t = 0.f;
#pragma unroll
                for (int j = 0; j < 8; ++j) t = fmaf(f[j], f[j], t);
                ss += tid + (k0 + k) * NT < d8 ? t : 0.f;
            }
            ss = wave_sum(ss);
            if ((tid & 63) == 0) nrm[wv * BT + b0 + r] = k0 > 0 ? nrm[wv * BT + b0 + r] + ss : ss;
        }
    };
    // (in front of the second weight batch: behind it the squares would wait for that batch; 16-row tile, 4 rows of
    // 4096: x staged at 10.3 us with the loads behind the batch)
    if (kLayer && !ROW) load_rows(0, 0);
    // the row that is the input of a stack with norm or residual, and the weights gamma that belong to it
    u32x4 rsl[2];
    uint4 grow;
    auto row_slots = [&]() {
        const size_t at = tid < d8 ? 4 * tid : 0;
        rsl[0] = xsl.ld2(at);
        rsl[1] = xsl.ld2(at + 2);
    };
    if constexpr (ROW) {
        grow = gg4[norm && tid < d8 ? tid : 0];
        if (from_slots)
            row_slots();
        else
            load_rows(0, 0);
    }
    // for the RoPE tables, below: the frequency and the position of every table entry of this thread
    constexpr int NE = RopeRows<HD, BT>::NE;
    const bool own_pos = kLayer && p.row_pos != nullptr;
    const int32_t *psrc = own_pos ? p.row_pos : reinterpret_cast<const int32_t *>(p.x);   // any readable address
    int epos[NE];
#pragma unroll
    for (int k = 0; k < NE; ++k) {
        const int e = tid + k * NT, eb = e / (HD / 2);
        epos[k] = psrc[own_pos && eb < p.B ? eb : 0];
    }
    if constexpr (kLayer && !STACK) lens = psrc[own_pos && (tid & 15) < p.B ? tid & 15 : 0];        // of row `lane % 16`, for deal_rows
    __builtin_amdgcn_sched_barrier(0);
    if (!(AHEAD >= 2 && primed)) load(wb, voff0);
    __builtin_amdgcn_sched_barrier(0);
    CF_STAMP(21);           // second weight batch issued
    // Launch number: every workgroup keeps, in a line of its own, the number of launches it has
    // completed; all workgroups of a launch hold the same count, so count + 1 stamps this launch
    // without any shared counter.  (One counter for all was read by 256 workgroups at once and
    // bumped by 256 atomics at the end: both are served one after the other, microseconds in all,
    // and the read sat at the head of the in-order return queue in front of the weights.)  The
    // value was written in an earlier launch, so a scalar load through the cache is good enough,
    // and it does not enter the vector memory queue at all.
    if (layer == 0) {
        unsigned long long launches;
        asm volatile("s_load_dwordx2 %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)"
                     : "=s"(launches)
                     : "s"(p.done + (size_t)blockIdx.x * kCounterStride)
                     : "memory");
        cnt0 = launches + 1ull;
    }
    const uint32_t stamp = stamp_of(cnt0, layer);
    // MF: the value goes to row b, column r of the operand array as fp16; without RMSNorm that is x itself, with it the product
    // x * gamma (22 bits), scaled by 2^xe and cut into a high and a low part, so that nothing is rounded away; the scale is
    // taken out with the row's factor.  (Without the scale the pair lost bits below one and was NaN above 65504: |x gamma|
    // 1e-2 / 1e-4 to 2e-6 / 2e-4 of the projected value.)
    int xe = 0;
    float xmax = 0.f;
    auto stage = [&](int i, int b, int r, float v) {
        if constexpr (MF)
            xh[b * XS + r] = (_Float16)v;
        else
            xs[i] = v;
    };
    // (rows past the batch are left as they are: what they give lands in rows of the product nobody reads)
    auto stage_piece = [&](int b, int c, const uint4 &xw, const uint4 &gw, bool in) {
        const h8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
        h8 hi = in ? __builtin_bit_cast(h8, xw) : zero;
        float f[8], g[8];
        unpack8(hi, f);
        if (norm) {
            unpack8(__builtin_bit_cast(h8, gw), g);
#pragma unroll
            for (int j = 0; j < 8; ++j) f[j] = in ? f[j] * g[j] : 0.f;
        }
        if constexpr (MF) {
            if (norm) {
                const mfma::Split<2> s = mfma::split_scaled<2>(f, xe, xmax);
                hi = s.part[0];
                *reinterpret_cast<h8 *>(xl + b * XS + 8 * c) = s.part[1];
            }
            *reinterpret_cast<h8 *>(xh + b * XS + 8 * c) = hi;
        } else {
            float *dst = xs + b * p.RPS + 8 * c;
            *reinterpret_cast<f32x4 *>(dst) = f32x4{f[0], f[1], f[2], f[3]};
            *reinterpret_cast<f32x4 *>(dst + 4) = f32x4{f[4], f[5], f[6], f[7]};
        }
    };
    // cos / sin of this position while x is still on its way (the same for every layer of a stack).  Behind the staged x it is at most 0.7 %
    // slower: us a pass, here / there, odd sizes at batch 3 32.5 / 32.6, 8192 columns, 4 heads, norm 33.9 / 34.1, 7B shape 70.2 / 70.2.
#pragma unroll
    for (int k = 0; k < NE; ++k) {
        const int e = tid + k * NT, eb = e / (HD / 2), i = e % (HD / 2);
        if (!STACK && eb < (own_pos ? p.B : 1)) {      // (a stack builds the table once, in front of its layers)
            const int pos_e = own_pos ? min(max(epos[k], 0), p.pos) : p.pos;
            // (the frequency is computed here: a table in memory was one more cold page in front of the first wait)
            rope_cos_sin(pos_e, rope_inv_freq(i, HD, p.rope_log2_base), rope[eb * HD + i], rope[eb * HD + HD / 2 + i]);
        }
    }
    // The slots carry the stamp of the previous layer.  A workgroup whose projection nobody waits for (no column block of its
    // own) may arrive here after its sources have moved on and stamped newer values: any stamp from the previous layer's up
    // to the last layer's of this launch is taken.
    const uint32_t want = stamp_of(cnt0, layer - 1);
    auto arrived = [&](uint32_t have) { return (uint32_t)(have - want) <= (uint32_t)n_layers; };
    if constexpr (ROW) {
        const int c = tid - (r0 >> 3), np = nrows >> 3;           // this thread's piece in the slice; pieces of the slice
        if (from_slots) {
            Spin spin;
            while (!((tid >= d8) | (arrived(rsl[0].y) & arrived(rsl[0].w) & arrived(rsl[1].y) & arrived(rsl[1].w)))) {
                if (spin.expired(p)) break;
                row_slots();
            }
            xq[0][0] = uint4{rsl[0].x, rsl[0].z, rsl[1].x, rsl[1].z};
        }
        if ((unsigned)c < (unsigned)np) stage_piece(0, c, xq[0][0], grow, true);
        if (norm) square_rows(0, 0);
        const uint4 none = {0u, 0u, 0u, 0u};
        for (int i = np + tid; i < P8; i += NT) stage_piece(0, i, none, none, false);     // the last slice may be shorter
    } else if constexpr (BYROW) {
        const bool live = brow < p.B;
        auto row_scale = [&]() {
            xmax = lpr == 32 ? lanes::max_half(xmax) : wave_max(xmax);
            xe = mfma::scale_exp(xmax);
        };
        auto take_max = [&](const uint4 &xw, const uint4 &gw, bool in) {
            float f[8], g[8];
            unpack8(__builtin_bit_cast(h8, xw), f);
            unpack8(__builtin_bit_cast(h8, gw), g);
#pragma unroll
            for (int j = 0; j < 8; ++j) f[j] *= g[j];
            const float m = mfma::max_abs(f, xmax);
            xmax = in ? m : xmax;
        };
        auto max_of_registers = [&]() {
#pragma unroll
            for (int q = 0; q < XP; ++q) {
                if (q * lpr >= P8) break;                         // (uniform)
                int b, c;
                const bool in = own_piece(q, b, c);
                take_max(xp[q], gp[q], in);
            }
        };
        auto stage_registers = [&]() {
#pragma unroll
            for (int q = 0; q < XP; ++q) {
                if (q * lpr >= P8) break;
                int b, c;
                const bool in = own_piece(q, b, c);
                if (live && c < P8) stage_piece(b, c, xp[q], norm ? gp[q] : xp[q], in);
            }
        };
        if (xvec && P8 <= XP * lpr) {                             // (uniform: all of a row's pieces are in registers)
            if (norm) {
                max_of_registers();
                row_scale();
            }
            stage_registers();
        } else if (xvec) {                                        // slices of more than 1024 (up to eight rows: 2048) values
            auto fetch = [&](const uint4 *src, size_t at, int c) { return src[8 * c < nrows ? at + r0 / 8 + c : 0]; };
            const size_t row8 = (size_t)brow * d8;
            if (norm) {
                max_of_registers();
                for (int c = lane0 + XP * lpr; live && c < P8; c += lpr) take_max(fetch(xg4, row8, c), fetch(gg4, 0, c), 8 * c < nrows);
                row_scale();
            }
            stage_registers();
            for (int c = lane0 + XP * lpr; live && c < P8; c += lpr) stage_piece(brow, c, fetch(xg4, row8, c), fetch(gg4, 0, c), 8 * c < nrows);
        } else {                                                  // slices that are no multiples of eight rows
            auto value = [&](int r) { return r < nrows ? h2f(p.x[(size_t)brow * p.D + r0 + r]) * (norm ? h2f(lp.gamma[r0 + r]) : 1.f) : 0.f; };
            if (norm) {
                for (int r = lane0; live && r < nrows; r += lpr) xmax = fmaxf(xmax, fabsf(value(r)));
                row_scale();
            }
            for (int r = lane0; live && r < p.RPS; r += lpr) {
                const float v = norm ? __builtin_amdgcn_ldexpf(value(r), xe) : value(r), hi = (float)__builtin_amdgcn_cvt_pkrtz(v, v)[0];
                xh[brow * XS + r] = (_Float16)hi;
                if (norm) xl[brow * XS + r] = (_Float16)(fabsf(v) <= 3.402823466e38f ? v - hi : 0.f);
            }
        }
    } else if (XV && xvec) {
#pragma unroll
        for (int q = 0; q < XP; ++q) {
            int b, c;
            const bool in = piece_of(tid + q * NT, b, c);
            if (tid + q * NT < npc) stage_piece(b, c, xp[q], norm ? gp[q] : xp[q], in);
        }
        for (int i = tid + XP * NT; i < npc; i += NT) {           // (16 rows: slices of more than 1024 values, 4 rows: of more than 2048)
            int b, c;
            const bool in = piece_of(i, b, c);
            stage_piece(b, c, xg4[in ? ((size_t)b * p.D + r0) / 8 + c : 0], gg4[in ? r0 / 8 + c : 0], in);
        }
    } else if constexpr (STACK) {
        auto take_pieces = [&](int i0) {                          // waits for the trip that starts at piece i0, and stages it
            if (from_slots) {
                Spin spin;
                for (;;) {
                    bool ok = true;
#pragma unroll
                    for (int q = 0; q < XP; ++q) {
                        int b, c;
                        ok &= !piece_of(i0 + tid + q * NT, b, c) |
                              (arrived(sp[q][0].y) & arrived(sp[q][0].w) & arrived(sp[q][1].y) & arrived(sp[q][1].w));
                    }
                    if (ok || spin.expired(p)) break;
                    piece_slots(i0);
                }
            }
#pragma unroll
            for (int q = 0; q < XP; ++q) {
                int b, c;
                const int i = i0 + tid + q * NT;
                const bool in = piece_of(i, b, c);
                const uint4 v = uint4{sp[q][0].x, sp[q][0].z, sp[q][1].x, sp[q][1].z};
                if (i < npc) stage_piece(b, c, v, v, in);
            }
        };
        // (the first trip outside the loop: inside it, its addresses are computed once more, 0.2 - 0.9 us a layer at batch 1)
        take_pieces(0);
        for (int trip = XP * NT; trip < npc; trip += XP * NT) {   // (uniform)
            int i0 = trip;
            asm volatile("" : "+s"(i0));                          // (the addresses of a trip are not kept for the next)
            if (from_slots)
                piece_slots(i0);
            else
                piece_values(i0);
            take_pieces(i0);
        }
    } else {
        for (int i = tid; i < xn; i += NT) {                      // (slices that are no multiples of eight rows)
            int b, r;
            const bool in = x_at(i, b, r);
            stage(i, b, r, in ? h2f(p.x[(size_t)b * p.D + r0 + r]) * (norm ? h2f(lp.gamma[r0 + r]) : 1.f) : 0.f);
        }
    }
    if (MF && !xvec) {
        // columns RPS .. XS-1 of every row: an operand read that starts inside the slice may reach up to seven columns past it
        // (with slices of 8 k rows it ends inside: nothing to clear when x came in pieces)
        const int nz = XS - p.RPS;
        for (int e = tid; e < 16 * nz; e += NT) {
            const int b = e / nz, r = p.RPS + (e - b * nz);
            xh[b * XS + r] = (_Float16)0.f;
            if (kLayer || HD == 128) xl[b * XS + r] = (_Float16)0.f;
        }
    }
    if (norm && !ROW) {
        square_rows(0, 0);
        for (int k0 = 0; k0 * NT < d8; k0 += KR)      // large batches: the other rows; long rows: their second half
            for (int b0 = k0 > 0 ? 0 : RG; b0 < p.B; b0 += RG) {
                load_rows(b0, k0);
                square_rows(b0, k0);
            }
    }
    lds_barrier();
    CF_STAMP(2);            // x staged

    float acc[MF ? 1 : BT][8];              // FMA tiles: [batch row][column] of this lane's row group
    // MFMA tiles: [row set][column][batch rows 4 * (lane / 16) + 0..3].  The columns of an operand share its rows of x, so every
    // set of x rows gets a product of its own with all the weights; a lane's sum is the one of its own set, the others are junk.
    f32x4 acc4[RS][MF ? 8 : 1];
#pragma unroll
    for (int b = 0; b < (MF ? 1 : BT); ++b)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[b][j] = 0.f;
#pragma unroll
    for (int c = 0; c < (MF ? 8 : 1) * RS; ++c) acc4[c % RS][c / RS] = f32x4{0.f, 0.f, 0.f, 0.f};
    int si_first = 0;                       // selector index of the first buffered item
    int nbuf = 0;
    bool factors = false;
    auto flush = [&]() {
        if (BYROW && norm && !factors && lane0 == 0 && brow < p.B) {          // the factor of a row, in the place of its first sum of squares
            float ss = 0.f;
#pragma unroll
            for (int w8 = 0; w8 < NW; ++w8) ss += nrm[w8 * BT + brow];
            nrm[brow] = __builtin_amdgcn_ldexpf(1.0f / sqrtf(ss / (float)p.D + p.eps), -xe);
        }
        factors = true;
        lds_barrier();
        for (int e = tid; e < nbuf * BT * HD; e += NT) {
            const int it = e / (BT * HD), rem = e - it * (BT * HD);
            const int b = rem / HD, c = rem - b * HD;
            if (b < p.B) {
                float sum = 0.f, ss = 0.f;
#pragma unroll
                for (int w8 = 0; w8 < NW; ++w8) sum += red[((it * NW + w8) * BT + b) * HD + c];
                if (BYROW) {
                    if (norm) sum *= nrm[b];
                } else if (norm) {
#pragma unroll
                    for (int w8 = 0; w8 < NW; ++w8) ss += nrm[w8 * BT + b];
                    sum *= 1.0f / sqrtf(ss / (float)p.D + p.eps);
                }
                x1.st((uint32_t)(ks * p.B + b) * p.nqkv + qkv_col0<HD, G>(p, team, sel_of(si_first + it)) + c, sum,
                      stamp);
            }
        }
        lds_barrier();
        nbuf = 0;
    };
    auto consume = [&](const h8(&w)[U]) {
        const int i0 = cc.i0;
        if constexpr (MF) {
            // one step of 32 rows: operand A = x[batch row lane % 16][rows of this lane's group], operands B =
            // the eight columns of this lane.  Rows past the slice: their weights are zero (past the end of the buffer)
            // and x, where an operand reaches them, is zero; a group that starts past the slice reads nothing.
            const h8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
            h8 f[8];
            transpose8(w, f);
#pragma unroll
            for (int h = 0; h < RS; ++h) {
                const int r = NG * i0 + 32 * (RS * wv + h) + 8 * kg;
                const int xo = (tid & 15) * XS + min(r, XS - 8);
                const h8 ah = r < nrows ? *reinterpret_cast<const h8 *>(xh + xo) : zero;
#pragma unroll
                for (int c = 0; c < 8; ++c) acc4[h][c] = mfma16(ah, f[c], acc4[h][c]);
                if (norm) {
                    const h8 al = r < nrows ? *reinterpret_cast<const h8 *>(xl + xo) : zero;
#pragma unroll
                    for (int c = 0; c < 8; ++c) acc4[h][c] = mfma16(al, f[c], acc4[h][c]);
                }
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                // a row past the slice has zero weights (past the end of the buffer) and any finite x
                const int r = min(grp + NG * (i0 + u), p.RPS - 1);
                float f[8];
                unpack8(w[u], f);
#pragma unroll
                for (int b = 0; b < BT; ++b) {
                    const float xv = xs[b * p.RPS + r];
#pragma unroll
                    for (int j = 0; j < 8; ++j) acc[b][j] = fmaf(xv, f[j], acc[b][j]);
                }
            }
        }
    };
    auto finish = [&]() {         // epilogue of the step just consumed, then move the cursor on
        const int si = cc.si, i0 = cc.i0;
        if (si >= nsel) return;                     // padding step: nothing was loaded
        advance(cc);
        if (i0 + U < iters) return;
        if constexpr (MF) {
            // last batch of this selector: the MFMA has already added the four row groups of the wavefront;
            // the lane holds eight adjacent columns of batch rows 4 * kg + 0..3
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float v[8];
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    v[c] = RS == 2 && rs ? acc4[RS - 1][c][r] : acc4[0][c][r];
                    if (RS == 2) v[c] += lanes::xor8(v[c]);             // the two row sets of a column
                }
                float *dst = red + ((nbuf * NW + wv) * BT + 4 * kg + r) * HD + lig * 8;
                if (rs == 0) {
                    *reinterpret_cast<f32x4 *>(dst) = f32x4{v[0], v[1], v[2], v[3]};
                    *reinterpret_cast<f32x4 *>(dst + 4) = f32x4{v[4], v[5], v[6], v[7]};
                }
            }
#pragma unroll
            for (int c = 0; c < 8 * RS; ++c) acc4[c % RS][c / RS] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (nbuf == 0) si_first = si;
            if (++nbuf == MAXI) flush();
        } else {
            // last batch of this selector: the row groups of a wavefront here, the wavefronts in flush(), in a fixed order
#pragma unroll
            for (int b = 0; b < BT; ++b) {
                float t[LPR / 8];
                lanes::fold8<LPR>(acc[b], t);
                float *dst = red + ((nbuf * NW + wv) * BT + b) * HD + lig * 8 + (tid & 63) / LPR * (LPR / 8);
#pragma unroll
                for (int j = 0; j < LPR / 8; ++j) dst[j] = t[j];
            }
#pragma unroll
            for (int b = 0; b < BT; ++b)
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[b][j] = 0.f;
            if (nbuf == 0) si_first = si;           // buffered items are consecutive selectors
            // (flushing as soon as the q heads are done, so that q leaves early, was measured: the two extra
            // barriers in the middle of the stream cost more than the early q gains)
            if (++nbuf == MAXI) flush();
        }
    };

    // Two steps are in flight at the top of every iteration.  The step count is padded to an even
    // number >= 2 (a padding step loads nothing and adds zeros), so that the loop body and the
    // tail are straight-line code with a fixed number of loads.  The scheduling barriers keep the
    // reload of a register batch behind its last use, so the batch stays in the same registers
    // (no branch may sit between consume() and the barrier: the multiply-adds would sink past it).
    const int nsteps2 = max(2, (nsteps + 1) & ~1);
    // the reload of a register batch must follow its last use, or the compiler keeps old and new
    // batch in different registers and copies them (after a full drain) at the end of every
    // iteration: the load offset is made to depend on the accumulators the batch was folded into
    auto after_consume = [&]() {
        uint32_t v = voff0;
        if constexpr (MF) {
#pragma unroll
            for (int c = 0; c < 8 * RS; ++c) asm volatile("" : "+v"(v) : "v"(acc4[c % RS][c / RS]));
        } else {
#pragma unroll
            for (int b = 0; b < BT; ++b)
                asm volatile("" : "+v"(v) : "v"(acc[b][0]), "v"(acc[b][1]), "v"(acc[b][2]), "v"(acc[b][3]),
                             "v"(acc[b][4]), "v"(acc[b][5]), "v"(acc[b][6]), "v"(acc[b][7]));
        }
        return v;
    };
    for (int k = 0; k + 2 < nsteps2; k += 2) {
        consume(wa);
        load(wa, after_consume());
        if (k == 0) CF_STAMP(16);       // first step consumed and reloaded
        finish();
        consume(wb);
        load(wb, after_consume());
        finish();
    }
    // tail: no step of this phase is left to issue, so the first loads of the next phase go out
    // before the last two steps are consumed.  (Not earlier: the partial-sum stores of the final
    // flush queue behind every load issued before them.)
    issue_next(0);
    consume(wa);
    finish();
    if (nsteps > 1) {       // (a padding step: small shapes have one step in all)
        consume(wb);
        finish();
    }
    if (nbuf) flush();
    return stamp;
}

// ---------------------------------------------------------------------------
// Phase 2: one (batch row, KV split) of the team's KV head, all G query heads
// (Alg. 3 steps 3-4; the new token is counted by the last split only).
// K/V rows are streamed in batches of U rows per row group, two batches in flight.
// ---------------------------------------------------------------------------
// The loads of the team's q partials are put in flight right behind this workgroup's own partial sums
// (at the end of phase 1, before the second part of the K/V prefetch) and checked when q is needed:
// where the other members were no later than this one, the sum costs no further round trip.  Covers
// value e = threadIdx.x of up to kEarly k-slices; anything else takes the polling path.
// (Eight in the one-launch stack, whose registers hold the next layer's weights too.  Of more slices nothing is requested: eight
// of ten cost a stack 1 - 4 % and could not be used; us a pass, eight requested / none: eight layers, 4096 columns, 8 heads, 512
// rows, 10 slices 123.5 / 120.9, 8 heads over 4, 2048 rows, 16 slices 144.6 / 138.9; sixteen of 21 in a single launch, 8192 columns, 4
// heads, two layers 34.6 / 32.6.)
template <int kEarly>
struct EarlyQ {
    static_assert(kEarly == 8 || kEarly == 16, "loads in groups of eight");
    u32x2 v[kEarly];
    bool issued = false;
    template <int HD, int G>
    __device__ __forceinline__ void issue(const Params &p, int tid0, int team, int b, int nsel)     // selectors to be summed
    {
        const Xbuf x1(p.p1);
        const int e = tid0;
        if (p.KS > kEarly) return;                        // (uniform)
        if (e < nsel * HD) {
            const int sel = e / HD, c = e - sel * HD;
            const uint32_t src = (uint32_t)(b * p.nqkv + qkv_col0<HD, G>(p, team, sel) + c);
            // eight loads at a time on a straight-line path (slices past KS repeat the last one)
            const uint32_t stride = (uint32_t)(p.B * p.nqkv);
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = x1.ld(src + (uint32_t)min(k, p.KS - 1) * stride);
            if (kEarly > 8 && p.KS > 8) {
#pragma unroll
                for (int k = 8; k < kEarly; ++k) v[k] = x1.ld(src + (uint32_t)min(k, p.KS - 1) * stride);
            }
        }
        issued = true;
    }
    // sum in slice order; false if a slot was not yet stamped or not covered
    __device__ __forceinline__ bool sum(const Params &p, uint32_t stamp, float &out) const
    {
        // (opaque: the sixteen comparisons with it would otherwise be made in front of the loop over the items and be kept)
        int n = p.KS;
        asm volatile("" : "+s"(n));
        uint32_t stale = issued ? 0u : 1u;
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            stale |= v[k].y ^ stamp;
            s += k < n ? __builtin_bit_cast(float, v[k].x) : 0.f;
        }
        if (kEarly > 8 && n > 8) {
#pragma unroll
            for (int k = 8; k < kEarly; ++k) {
                stale |= v[k].y ^ stamp;
                s += k < n ? __builtin_bit_cast(float, v[k].x) : 0.f;
            }
        }
        out = s;
        return stale == 0;
    }
};

// Selectors an attention item sums before it starts: its query heads, and for the item with the new token the new key and value
// too, where the threads suffice for all of them in one trip.  (Behind the cached rows that trip and two barriers are the end of
// the longest item.)  Us a layer, behind / first: tiny shape 13.9 / 13.4, 32 heads of 64, batch 12 30.4 / 30.0, Llama-2-7B shape 37.2 / 36.7; at
// head_dim 128 with more rows or heads the queries wait for it: batch 2 / 8, 16 heads 21.6 / 21.8, 25.6 / 26.0, two heads per group,
// batch 1 / 16 19.4 / 19.7, 37.0 / 37.9.
template <int HD, int G, int BT>
struct NewTokenFirst {
    static constexpr bool on = (G + 2) * HD <= NT && (HD == 64 || (G == 1 && BT == 1));
    static __device__ __forceinline__ int selectors(bool last) { return on && last ? G + 2 : G; }
};

template <int G>
struct P2Cfg {
    static constexpr int U = G >= 4 ? 2 : 4;    // rows per row group in one batch of loads
    static constexpr int GP = G >= 4 ? 4 : G;   // query heads handled per pass over a batch
    static constexpr int NB = 2;                // batches in flight
};

// Attention on MFMA tiles (head_dim 128, four or more query heads per KV head): the G query heads that share
// a K/V row are the (zero-padded) 16-row edge of two dense products per 32 cached tokens,
//   S^T = K q^T   (A = K rows, B = q, contraction over head_dim in four steps of 32),
//   O  += P V     (A = P, B = V, contraction over the 32 tokens),
// in place of 16 G multiply-adds per loaded 16 bytes on the vector ALU, which is what bounds the plain loop
// from G = 4 on.  A wavefront owns every eighth tile of 32 tokens of the split.  K rows are loaded row by
// row (16 lanes x 16 bytes), put into a tile of LDS that only this wavefront uses and read back as A operands
// (lane l: token l % 16, eight of the 32 dimensions of a step); the result has token 4 (l / 16) + r of each
// 16-token half in register r of lane (head l % 16).  Those eight scores of a lane are, after the softmax,
// exactly the lane's A operand of the second product if contraction index (l / 16, e) stands for token
// 16 (e / 4) + 4 (l / 16) + e % 4, so V rows are loaded in that order and transposed in the lane
// (transpose8), and nothing moves between the two products.
template <int HD, int G>
struct AttnMfma {
    static constexpr bool on = HD == 128 && G >= 4;
    static constexpr int kTile = 32;                   // tokens per tile
    static constexpr int kRowH = HD + 8;               // halves per K row in LDS (16 bytes of padding: bank spread)
    static constexpr int kTileFloats = kTile * kRowH / 2;   // LDS floats per wavefront
};

template <int HD, int G>
struct KvBuf {
    static constexpr bool MA = AttnMfma<HD, G>::on;
    static constexpr int NBd = MA ? 1 : P2Cfg<G>::NB, Ud = MA ? 8 : P2Cfg<G>::U;
    h8 k[NBd][Ud], v[NBd][Ud];
};

template <int HD, int G>
struct P2Stream {
    static constexpr int LPR = HD / 8;
    static constexpr int NG = NT / LPR;
    static constexpr int U = P2Cfg<G>::U;
    static constexpr bool MA = AttnMfma<HD, G>::on;
    int t0, t1, iters, grp, pos, tid;
    uint32_t voff0;          // of the lane's first row of the split
    size_t head;
    Stream K, V;
    // `pos_b`: tokens cached for this batch row, [t0, t1) the split.  The buffers end with the split: rows behind it, and so rows
    // >= pos_b, are never read.
    __device__ __forceinline__ P2Stream(const Params &p, const LayerPtrs &lp, int tid0, int team, int b, int t0_, int t1_, int pos_b)
        : t0(t0_), t1(t1_), grp(tid0 / LPR), pos(pos_b), tid(tid0), head(((size_t)b * p.nkv + team) * p.max_seq * HD),
          K(lp.kc + head, (uint32_t)t1 * HD * 2), V(lp.vc + head, (uint32_t)t1 * HD * 2)
    {
        const int n = max(t1 - t0, 0);
        iters = MA ? (n + 32 * NW - 1) / (32 * NW) : (n + NG - 1) / NG;   // MA: rounds of one 32-token tile per wavefront
        voff0 = (uint32_t)(t0 + grp) * HD * 2 + tid % LPR * 16;
    }
    // Split s of the plan.  An inactive stream (a workgroup without an attention item) has an empty split; a row shorter than the
    // longest one of the batch uses the same split boundaries: its splits past pos_b are empty.
    static __device__ __forceinline__ P2Stream planned(const Params &p, const LayerPtrs &lp, int tid0, int team, int b, int s, int pos_b, bool active = true)
    {
        const int first = s * p.TPS + ((s & 1) ? p.TD : 0);               // even splits are 2*TD tokens longer
        return P2Stream(p, lp, tid0, team, b, first, active ? min(first + p.TPS + ((s & 1) ? -p.TD : p.TD), pos_b) : 0, pos_b);
    }
    // MFMA tiles: round `it` gives wavefront wv the tokens t0 + 32 (8 it + wv) + 0..31.  K: load u brings rows
    // 4 u + (lane / 16); V: load u brings rows 16 (u / 4) + 4 (lane / 16) + u % 4 (the order in which the scores
    // come out of the first product).  Eight load instructions each.
    __device__ __forceinline__ void load_k(h8 (&kr)[8], int it, uint32_t dep) const
    {
        const int wv = tid >> 6, rg = (tid & 63) >> 4, lig = tid & 15;
        const uint32_t off = (uint32_t)(t0 + 32 * (NW * it + wv) + rg) * HD * 2 + lig * 16 + dep;
#pragma unroll
        for (int u = 0; u < 8; ++u) kr[u] = K.ld(off + 4 * u * HD * 2);
    }
    __device__ __forceinline__ void load_v(h8 (&vr)[8], int it, uint32_t dep) const
    {
        const int wv = tid >> 6, rg = (tid & 63) >> 4, lig = tid & 15;
        const uint32_t off = (uint32_t)(t0 + 32 * (NW * it + wv) + 4 * rg) * HD * 2 + lig * 16 + dep;
#pragma unroll
        for (int u = 0; u < 8; ++u) vr[u] = V.ld(off + (16 * (u >> 2) + (u & 3)) * HD * 2);
    }
    // Always 2*U load instructions on a straight-line path,
    // so that the compiler's wait counts for earlier loads stay exact.
    __device__ __forceinline__ void load(h8 (&kr)[U], h8 (&vr)[U], int i0, uint32_t voff) const
    {
        const uint32_t off = voff + (uint32_t)(NG * i0) * HD * 2;
#pragma unroll
        for (int u = 0; u < U; ++u) kr[u] = K.ld(off + (uint32_t)(NG * u) * HD * 2);
#pragma unroll
        for (int u = 0; u < U; ++u) vr[u] = V.ld(off + (uint32_t)(NG * u) * HD * 2);
        // (the order of the batches is kept: where a later one is requested first, the loop waits for all of them)
        __builtin_amdgcn_sched_barrier(0);
    }
    // the first NB batches do not depend on q: they are put in flight before q is needed; part 0
    // (two batches) before the last steps of phase 1, part 1 (the rest) once phase 1 has stored
    // its partial sums (stores queue behind every load issued before them)
    __device__ __forceinline__ void prefetch(KvBuf<HD, G> &buf, int part) const
    {
        constexpr int NB = P2Cfg<G>::NB;
        if constexpr (MA) {
            if (part == 0)
                load_k(buf.k[0], 0, 0u);
            else
                load_v(buf.v[0], 0, 0u);
        } else {
#pragma unroll
            for (int j = 0; j < NB; ++j)
                if ((j < 2) == (part == 0)) load(buf.k[j], buf.v[j], j * U, voff0);
        }
    }
};

template <int HD, int G, int BT, class Early, class TailFn>
__device__ __forceinline__ void p2_item(const Params &p, const LayerPtrs &lp, int tid0, int team, int b, int s, int ns, int row_item, uint32_t stamp, bool first,
                                        const P2Stream<HD, G> &st, KvBuf<HD, G> &buf, const Early &eq, float *smem,
                                        const float *rope, TailFn &&issue_next)
{
    constexpr int LPR = HD / 8;
    constexpr int NG = NT / LPR;
    constexpr int U = P2Cfg<G>::U;
    constexpr int NB = P2Cfg<G>::NB;
    constexpr int PS = HD + kP2Stride;
    // (the thread index is made opaque per item: everything derived from it would otherwise be computed once in
    // front of the loop over the items, dozens of registers that are then spilled)
    int tid = tid0;
    if (AttnMfma<HD, G>::on) asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wv = tid >> 6, lig = tid % LPR, grp = tid / LPR;
    const bool last = (s == ns - 1);             // of the row's ns splits, whose first is item `row_item`
    const Xbuf x1(p.p1);

    const float *cs = rope;                 // [HD/2] cos, filled at kernel start
    const float *sn = rope + HD / 2;        // [HD/2] sin
    float *qs = smem;                       // [G][HD]
    float *kn = qs + G * HD;                // [HD] rotated new key
    float *vn = kn + HD;                    // [HD] new value
    float *snew = vn + HD;                  // [8]  scores of the new token, log2 domain
    constexpr bool MA = AttnMfma<HD, G>::on;                    // both products on MFMA tiles
    constexpr int NPART = NW;               // partials that are folded through LDS: one per wavefront
    float *redm = snew + 8;                 // [G][NPART]
    float *redl = redm + G * NPART;         // [G][NPART]
    float *redacc = redl + G * NPART;       // [G][NPART][HD]
    const int t0 = st.t0, t1 = st.t1, iters = st.iters;

    // ---- sum the projection partials of the team (the gather of Alg. 3 step 3): q heads, and for
    //      the last split also the new key and value; then RoPE on q and the key
    constexpr bool KVF = NewTokenFirst<HD, G, BT>::on;              // the new key and value beside the queries (kn and vn follow qs)
    const int nsel = NewTokenFirst<HD, G, BT>::selectors(last);
    for (int e = tid; e < nsel * HD; e += NT) {
        const int sel = e / HD, c = e - sel * HD;
        const uint32_t src = (uint32_t)(b * p.nqkv + qkv_col0<HD, G>(p, team, sel) + c);
        float v;
        if (!(first && e == tid && eq.sum(p, stamp, v)))
            v = ll_sum(p, x1, src, (uint32_t)(p.B * p.nqkv), p.KS, stamp);
        qs[e] = v;
    }
    lds_barrier();
    for (int e = tid; e < min(nsel, G + 1) * (HD / 2); e += NT) {          // (not the value)
        const int sel = e / (HD / 2), i = e - sel * (HD / 2);
        float *v = qs + sel * HD;
        const float lo = v[i], hi = v[i + HD / 2], c = cs[i], sgn = sn[i];
        v[i] = lo * c - hi * sgn;
        v[i + HD / 2] = hi * c + lo * sgn;
    }
    lds_barrier();
    // q fragments of this lane's 8 columns, pre-scaled by log2(e)/sqrt(d).  Up to GP heads stay in
    // registers; wider groups (G > GP) re-read them from LDS for every pass over a batch.
    constexpr int GP = P2Cfg<G>::GP;
    constexpr bool kQsScaled = !MA && G > GP;                   // qs is overwritten by the scaled q
    float qf[GP][8];
    if constexpr (MA) {
        constexpr int RH = AttnMfma<HD, G>::kRowH;
        _Float16 *kt = reinterpret_cast<_Float16 *>(redacc + G * NPART * HD) + wv * (AttnMfma<HD, G>::kTile * RH);
        const int hq = lane & 15, quad = lane >> 4;             // operand row / column of the lane, contraction group
        // B operands of K q^T: head hq (zero for hq >= G), the lane's eight of the 32 dimensions of each step,
        // pre-scaled by log2(e)/sqrt(d), as high + low fp16 parts so that q keeps its fp32 bits.  They are the
        // same for every wavefront and every tile: kept in LDS ([step][lane], high then low), not in registers.
        h8 *qop = reinterpret_cast<h8 *>(redacc + G * NPART * HD + NW * AttnMfma<HD, G>::kTileFloats);
        if (tid < 256) {
            const int s4 = tid >> 6;
            float a[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) a[e] = hq < G ? qs[hq * HD + 32 * s4 + 8 * quad + e] * p.qk_scale_log2e : 0.f;
            h8 hi, lo;
            split_hi_lo(a, hi, lo);
            qop[tid] = hi;
            qop[256 + tid] = lo;
        }
        lds_barrier();
        CF_STAMP(14);           // q ready
        float m = kNegBig, l = 0.f;      // of head hq: running maximum (the same in the four lanes of a head), sum of this lane's tokens
        f32x4 O[8];                      // [column of the lane][heads 4 quad + 0..3]
#pragma unroll
        for (int c = 0; c < 8; ++c) O[c] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int it = 0; it < st.iters; ++it) {
            // ---- K rows -> this wavefront's tile in LDS -> A operands; the registers are reloaded at once
#pragma unroll
            for (int u = 0; u < 8; ++u) *reinterpret_cast<h8 *>(kt + (4 * u + quad) * RH + lig * 8) = buf.k[0][u];
            __builtin_amdgcn_sched_barrier(0);
            st.load_k(buf.k[0], it + 1, 0u);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            f32x4 S[2];
#pragma unroll
            for (int T = 0; T < 2; ++T) {
                S[T] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s4 = 0; s4 < 4; ++s4) {
                    const h8 kf = *reinterpret_cast<const h8 *>(kt + (16 * T + hq) * RH + 32 * s4 + 8 * quad);
                    S[T] = mfma16(kf, qop[s4 * 64 + lane], S[T]);
                    S[T] = mfma16(kf, qop[256 + s4 * 64 + lane], S[T]);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            // ---- online softmax of head hq over the lane's eight tokens 16 T + 4 quad + r
            const int tb = t0 + 32 * (NW * it + wv) + 4 * quad;
            float sc[8];
            bool ok[8];
            float mx = kNegBig;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                ok[e] = tb + 16 * (e >> 2) + (e & 3) < t1;
                sc[e] = ok[e] ? S[e >> 2][e & 3] : kNegBig;
                mx = fmaxf(mx, sc[e]);
            }
            mx = fmaxf(mx, __shfl_xor(mx, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float mn = fmaxf(m, mx);
            if (__any(mn > m)) {
                // a maximum has grown (rare after the first tiles): rescale the sum and the accumulators; the lane
                // holds heads 4 quad + r, whose factors are in lanes 4 quad + r
                const float scale = __builtin_amdgcn_exp2f(m - mn);
                l *= scale;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float sr = __shfl(scale, 4 * quad + r);
#pragma unroll
                    for (int c = 0; c < 8; ++c) O[c][r] *= sr;
                }
                m = mn;
            }
            float pv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                pv[e] = ok[e] ? __builtin_amdgcn_exp2f(sc[e] - mn) : 0.f;
                l += pv[e];
            }
            h8 ph, pl;
            split_hi_lo(pv, ph, pl);
            // ---- O += P V
            h8 f[8];
            transpose8(buf.v[0], f);
            __builtin_amdgcn_sched_barrier(0);
            st.load_v(buf.v[0], it + 1, 0u);
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                O[c] = mfma16(ph, f[c], O[c]);
                O[c] = mfma16(pl, f[c], O[c]);
            }
        }
        CF_STAMP(15);           // K/V consumed
        if (!last) issue_next(1);
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        if (hq < G && quad == 0) {
            redm[hq * NPART + wv] = m;
            redl[hq * NPART + wv] = l;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int g = 4 * quad + r;
            if (g < G) {
                float *dst = redacc + (g * NPART + wv) * HD + lig * 8;
                *reinterpret_cast<f32x4 *>(dst) = f32x4{O[0][r], O[1][r], O[2][r], O[3][r]};
                *reinterpret_cast<f32x4 *>(dst + 4) = f32x4{O[4][r], O[5][r], O[6][r], O[7][r]};
            }
        }
    } else {
    if (G > GP) {
        for (int e = tid; e < G * HD; e += NT) qs[e] *= p.qk_scale_log2e;   // qs now holds the scaled q
        lds_barrier();
    } else {
#pragma unroll
        for (int g = 0; g < GP; ++g)
#pragma unroll
            for (int j = 0; j < 8; ++j) qf[g][j] = qs[g * HD + lig * 8 + j] * p.qk_scale_log2e;
    }
    CF_STAMP(14);           // q ready

    // ---- online softmax over this split's cached tokens; one row per LPR lanes
    float m[G], l[G], acc[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        m[g] = kNegBig;
        l[g] = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[g][j] = 0.f;
    }
    auto consume = [&](const h8(&kr)[U], const h8(&vr)[U], int i0) {
#pragma unroll
        for (int g0 = 0; g0 < G; g0 += GP) {
            if (G > GP) {
#pragma unroll
                for (int g = 0; g < GP; ++g)
#pragma unroll
                    for (int j = 0; j < 8; ++j) qf[g][j] = qs[(g0 + g) * HD + lig * 8 + j];
            }
            float sc[GP][U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float kf[8];
                unpack8(kr[u], kf);
                const bool ok = (t0 + grp + NG * (i0 + u)) < t1;
#pragma unroll
                for (int g = 0; g < GP; ++g) {
                    float d = 0.f;
#pragma unroll
                    for (int j = 0; j < 8; ++j) d = fmaf(qf[g][j], kf[j], d);
                    d = row_sum<LPR>(d);
                    sc[g][u] = ok ? d : kNegBig;
                }
            }
            float pr[GP][U];
#pragma unroll
            for (int g = 0; g < GP; ++g) {
                float mn = m[g0 + g];
#pragma unroll
                for (int u = 0; u < U; ++u) mn = fmaxf(mn, sc[g][u]);
                const float scale = __builtin_amdgcn_exp2f(m[g0 + g] - mn);
                m[g0 + g] = mn;
                float ls = l[g0 + g] * scale;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const bool ok = (t0 + grp + NG * (i0 + u)) < t1;
                    pr[g][u] = ok ? __builtin_amdgcn_exp2f(sc[g][u] - mn) : 0.f;
                    ls += pr[g][u];
                }
                l[g0 + g] = ls;
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[g0 + g][j] *= scale;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float vf[8];
                unpack8(vr[u], vf);
#pragma unroll
                for (int g = 0; g < GP; ++g)
#pragma unroll
                    for (int j = 0; j < 8; ++j) acc[g0 + g][j] = fmaf(pr[g][u], vf[j], acc[g0 + g][j]);
            }
        }
    };
    // NB batches are in flight at the top of every iteration.  The reload offset is made to depend on the state the batch was
    // folded into: the reload then follows the last use of the registers it overwrites, so no copy and no drain is needed.  The
    // last NB batches are folded behind the loop: a reload with nothing to load would still have to return, behind everything
    // requested before it, before its registers can be used again, and a short split has one batch in all.
    auto after_consume = [&]() {
        uint32_t v = st.voff0;
#pragma unroll
        for (int g = 0; g < G; ++g)
            asm volatile("" : "+v"(v) : "v"(acc[g][0]), "v"(acc[g][1]), "v"(acc[g][2]), "v"(acc[g][3]),
                         "v"(acc[g][4]), "v"(acc[g][5]), "v"(acc[g][6]), "v"(acc[g][7]), "v"(l[g]), "v"(m[g]));
        return v;
    };
    static_assert(NB == 2, "two batches behind the loop");
    int i0 = 0;
    for (; i0 + NB * U < iters; i0 += NB * U) {
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            consume(buf.k[j], buf.v[j], i0 + j * U);
            __builtin_amdgcn_sched_barrier(0);
            st.load(buf.k[j], buf.v[j], i0 + (j + NB) * U, after_consume());
        }
    }
    if (i0 < iters) consume(buf.k[0], buf.v[0], i0);
    if (i0 + U < iters) consume(buf.k[1], buf.v[1], i0 + U);
    CF_STAMP(15);           // K/V consumed
    // Nothing of this phase is left to load.  Half of the next phase's first tile goes out now and
    // streams while the partial is merged and stored; the other half follows the stored partial.
    // (Not all of it now: the vector memory path of a compute unit returns in order, so the stamped
    // store and the next phase's polls wait for every bulk load issued before them.)  The member with
    // the last split first polls for the new token's key/value sums, for the same reason, where it has not done so yet.
    if (!last || KVF) issue_next(1);
    // ---- merge the row groups of a wavefront
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const float mw = lanes::max_groups<LPR>(m[g]), f = __builtin_amdgcn_exp2f(m[g] - mw);
        const float lw = lanes::sum_groups<LPR>(l[g] * f);
        if (lane == 0) {
            redm[g * NPART + wv] = mw;
            redl[g * NPART + wv] = lw;
        }
        float t[LPR / 8];
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[g][j] *= f;
        lanes::fold8<LPR>(acc[g], t);
        float *dst = redacc + (g * NPART + wv) * HD + lig * 8 + lane / LPR * (LPR / 8);
#pragma unroll
        for (int j = 0; j < LPR / 8; ++j) dst[j] = t[j];
    }
    }   // !MA
    CF_STAMP(8);            // row groups of the wavefront merged
    if (last) {
        // ---- the new token: sum its key/value partials (stored at the end of phase 1, long ago by
        //      now), rotate the key, append both (Sec. 2.1) and score the token
        if constexpr (!KVF) {
            for (int e = tid; e < 2 * HD; e += NT) {
                const int sel = G + e / HD, c = e % HD;
                const uint32_t src = (uint32_t)(b * p.nqkv + qkv_col0<HD, G>(p, team, sel) + c);
                kn[e] = ll_sum(p, x1, src, (uint32_t)(p.B * p.nqkv), p.KS, stamp);      // kn and vn are contiguous
            }
            issue_next(1);
            lds_barrier();
            if (tid < HD / 2) {
                const float lo = kn[tid], hi = kn[tid + HD / 2], c = cs[tid], sgn = sn[tid];
                kn[tid] = lo * c - hi * sgn;
                kn[tid + HD / 2] = hi * c + lo * sgn;
            }
            lds_barrier();
        }
        const size_t row = st.head + (size_t)st.pos * HD;
        if (tid < HD)
            lp.kc[row + tid] = f2h(kn[tid]);
        else if (tid < 2 * HD)
            lp.vc[row + tid - HD] = f2h(vn[tid - HD]);
        for (int g = wv; g < G; g += NW) {
            float d = 0.f;
            for (int c = lane; c < HD; c += 64) d = fmaf(qs[g * HD + c], kn[c], d);
            d = wave_sum(d);
            if (lane == 0) snew[g] = kQsScaled ? d : d * p.qk_scale_log2e;
        }
        if (p.dbg_q)
            for (int e = tid; e < G * HD; e += NT)
                p.dbg_q[((size_t)b * p.nq + team * G) * HD + e] =
                    kQsScaled ? qs[e] / p.qk_scale_log2e : qs[e];
    }
    lds_barrier();
    CF_STAMP(9);            // new token handled, wavefronts in step
    // ---- the wavefronts and the new token -> one partial (m, l, acc) per query head
    const Xbuf x2(p.p2);
    for (int e = tid; e < G * HD; e += NT) {
        const int g = e / HD, c = e - g * HD;
        float M = last ? snew[g] : kNegBig;
#pragma unroll
        for (int w8 = 0; w8 < NPART; ++w8) M = fmaxf(M, redm[g * NPART + w8]);
        float L = 0.f, A = 0.f;
#pragma unroll
        for (int w8 = 0; w8 < NPART; ++w8) {
            const float f = __builtin_amdgcn_exp2f(redm[g * NPART + w8] - M);
            L = fmaf(redl[g * NPART + w8], f, L);
            A = fmaf(redacc[(g * NPART + w8) * HD + c], f, A);
        }
        if (last) {
            const float f = __builtin_amdgcn_exp2f(snew[g] - M);
            L += f;
            A = fmaf(vn[c], f, A);
        }
        const uint32_t dst = (uint32_t)((row_item * p.nq + (team * G + g) * ns + s) * PS);
        if (c == 0) {
            x2.st(dst, M, stamp);
            x2.st(dst + 1, L, stamp);
        }
        x2.st(dst + kP2Stride + c, A, stamp);
    }
    CF_STAMP(10);            // partial stored
    issue_next(2);       // the rest of the tile, behind the stored partial
    lds_barrier();
}

// ---------------------------------------------------------------------------
// Phase 3: merge the split-KV partials of head hq (Alg. 3 steps 5-7), multiply by
// rows [rs*n, (rs+1)*n), n = HD >> LRS3, x columns [c3*CW3, (c3+1)*CW3) of that head's
// W_o block (step 8) and leave a per-head partial of the output.  The first
// 512-column chunk is loaded into registers before the attention result is needed.
// ---------------------------------------------------------------------------
template <int HD>
struct OutTile {
    static constexpr int MAXR = HD / 8;    // 16-byte loads per thread when a head is not split over rows
    h8 w[MAXR];
};

// Chunk `ch` of an item of the output projection: its rows of W_o as a buffer, and the lane's place in it.  Vector tiles:
// wavefront wv takes 64 columns of the chunk, its eight row groups of eight lanes the rows r + 8 u.  MF (MFMA tiles): wavefront wv
// takes columns [128 (wv % 4), +128) of the chunk and one half of the head's HD rows (wv / 4); lane (l % 16, l / 16) loads eight
// adjacent columns of rows 32 s + 8 (l / 16) + 0..7 for the steps s (one or two; the same lane layout as in the projection: eight
// rows are transposed in the lane into MFMA operands).  Lanes past the last column load nothing.
template <int HD, bool MF>
struct OutRows {
    Stream W;
    uint32_t off, rowb;
    __device__ __forceinline__ OutRows(const Params &p, const LayerPtrs &lp, int tid, int hq, int c3, int rs, int ch, bool live)
        : W(reinterpret_cast<const char *>(lp.wo) + (size_t)(uint32_t)hq * p.ohead +
                (size_t)(uint32_t)((HD >> p.LRS3) * rs * p.orow + ((c3 * p.CW3 + ch * kOutChunk) / kOutChunk) * p.ochunk),
            live ? (uint32_t)((HD >> p.LRS3) - 1) * p.orow + min(kOutChunk, p.D - c3 * p.CW3 - ch * kOutChunk) * 2u : 0u),
          rowb(p.orow)
    {
        const int lane = tid & 63, wv = tid >> 6;
        const int row = MF ? HD / 2 * (wv >> 2) + 8 * (lane >> 4) : lane >> 3, col = MF ? 128 * (wv & 3) + 8 * (lane & 15) : 64 * wv + 8 * (lane & 7);
        off = c3 * p.CW3 + ch * kOutChunk + col < p.D ? (uint32_t)row * rowb + col * 2 : kNoLoad;
        // (opaque to the compiler: it otherwise computes the sixteen per-row offsets of all call sites once, far
        // ahead of the first one, and spills them)
        asm volatile("" : "+v"(off));
    }
    __device__ __forceinline__ h8 row(int u, uint32_t at) const { return W.ld(at + (uint32_t)(MF ? 32 * (u >> 3) + (u & 7) : 8 * u) * rowb); }
};

// part: 0 = first half of the tile's loads, 1 = second half, 2 = all
template <int HD, bool MF>
__device__ __forceinline__ void p3_load(const Params &p, const LayerPtrs &lp, int tid, int hq, int c3, int rs, int ch, OutTile<HD> &t, int part = 2,
                                        bool live = true)
{
    const OutRows<HD, MF> o(p, lp, tid, hq, c3, rs, ch, live);
#pragma unroll
    for (int u = 0; u < OutTile<HD>::MAXR; ++u) {
        if (part == 2 || (part == 0) == (u < OutTile<HD>::MAXR / 2)) t.w[u] = o.row(u, o.off);
    }
}

template <int HD, int BT, int MCW>
__device__ __forceinline__ void p3_item(const Params &p, const LayerPtrs &lp, int tid0, int hq, int c3, int rs, uint32_t stamp, OutTile<HD> &tile,
                                        float *smem, const int *row_items)
{
    constexpr int PS = HD + kP2Stride;
    // (the thread index is made opaque here, so that what this phase derives from it is computed here and not kept from the start
    // of the kernel or, in front of the loop over the items, for all of them)
    int tid = tid0;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wv = tid >> 6;
    // merged, normalised attention output of head hq, [BT][HD].  MFMA tiles: as operands, PARTS fp16 parts [16][AR] of every
    // value, and what undoes their scale, [16][2] (64 columns each).  (Unpadded rows would be read from the same LDS
    // banks: Llama-3-8B shape, batch 4, 1.8 us for a product of 0.3.)
    constexpr bool MF = Mfma<HD, BT>::on;
    constexpr int AR = HD + kOutPad, PARTS = out_parts(HD);
    float *as = smem;
    _Float16 *ap = reinterpret_cast<_Float16 *>(smem);
    float *inv = smem + PARTS * 16 * AR / 2;
    float *red = smem + (MF ? out_operand_floats(HD) : BT * HD);          // the sums of the merge; MFMA tiles: [2][16][512]
    const Xbuf x2(p.p2), x3(p.p3);

    const int nrows = HD >> p.LRS3;
    const int rbeg = rs * nrows;
    const int iters = nrows / 8;
    const int slot = (hq << p.LRS3) + rs;
    const int nchunk = p.CW3 / kOutChunk;

    {
        // ---- merge of the split-KV partials (Alg. 3 steps 5-7).  A pass handles up to NV * 512 values v = (batch row,
        //      column).  NV == 1: value v is handled by SG threads, each adding every SG-th split; the SG sums are then
        //      added through LDS.  NV > 1 (more values than threads): a thread adds all splits of NV values.  The maxima
        //      and sums of a row's splits are fetched once per wavefront (a wavefront's values belong to one batch row):
        //      lane s holds those of split s and, after two reductions over the wavefront, its weight e^(m_s - M) / L.
        //      All loads of a round go out together, MC splits per round trip.  (Fetched by every thread beside each
        //      value they were two thirds of the loads: tiny shape 17.2 -> 15.5 us, Llama-3-8B shape at batch 8 67.4 -> 65.9 us, 3000
        //      columns at batch 5 29.1 -> 27.2 us; a branch around the loads past the last split costs more than they do.)
        const int V = p.B * HD;
        // value vi of the wavefront's 64, neighbours in one row.  MFMA tiles: scaled by a power of two that brings the largest of
        // them into [2^14, 2^15) and split into fp16 parts, so that they enter the product with the same bits whatever their
        // magnitude (an unscaled pair: 1e-2 of the output at 1e-6)
        constexpr int kNoScale = -114;                            // an infinity among them
        auto scale_of = [&](int max_bits) { return min(141 - (max_bits >> 23), 126); };
        auto keep = [&](int vi, float v, int e) {
            const int b = vi / HD, c = vi - b * HD;
            if constexpr (MF) {
                float r = __builtin_amdgcn_ldexpf(v, e);
#pragma unroll
                for (int n = 0; n < PARTS; ++n) {
                    const _Float16 t = (_Float16)r;
                    ap[(n * 16 + b) * AR + c] = t;
                    r = e == kNoScale ? 0.f : r - (float)t;       // (an infinity stays one, in the first part)
                }
                if (lane == 0) inv[2 * b + c / 64] = __builtin_bit_cast(float, (127 - e) << 23);
            } else {
                as[vi] = v;
            }
            if (p.dbg_attn && c3 == 0 && rs == 0) p.dbg_attn[((size_t)b * p.nq + hq) * HD + c] = v;
        };
        auto run = [&](auto nv_c, auto mc_c, auto ragged_c) {
            constexpr int NV = decltype(nv_c)::value, MC = decltype(mc_c)::value;
            constexpr bool ragged = decltype(ragged_c)::value;            // the rows' splits by the table (an instance of its own: 0.3 us a layer)
            for (int v0 = 0; v0 < V; v0 += NT * NV) {
                const int cv = min(NT * NV, V - v0);                      // a multiple of 64
                const float rcv = reciprocal(cv);
                const int SG = NV == 1 ? max(1, min(__builtin_amdgcn_readfirstlane(fdiv(NT, rcv)), ragged ? p.TS : p.NS)) : 1;
                const int sg = NV == 1 ? __builtin_amdgcn_readfirstlane(fdiv(tid, rcv)) : 0, v = tid - sg * cv;
                if (sg < SG) {
                    float at[NV], wgt[NV];
                    uint32_t src[NV];
                    int col[NV], ns[NV], most = ragged ? 1 : p.NS;    // splits of the value's row; most of them
#pragma unroll
                    for (int n = 0; n < NV; ++n) {
                        at[n] = 0.f;
                        wgt[n] = 0.f;
                        const int vi = min(v0 + v + n * NT, V - 1);        // a value past the end repeats the last one
                        const int b = vi / HD;
                        col[n] = vi - b * HD;
                        ns[n] = p.NS;
                        int row_item = b * p.NS;
                        if constexpr (ragged) {
                            row_item = __builtin_amdgcn_readfirstlane(row_items[b]);
                            ns[n] = __builtin_amdgcn_readfirstlane(row_items[b + 1]) - row_item;
                        }
                        if (ragged) most = max(most, ns[n]);
                        src[n] = (uint32_t)((row_item * p.nq + hq * ns[n]) * PS);
                    }
                    const bool wide = most > 32;                          // more splits than half a wavefront: two loads
                    for (int sb = sg; sb < most; sb += MC * SG) {
                        const bool head = sb == sg;                       // the first round
                        Spin spin;
                        u32x2 vm[NV], vl[NV], va[NV][MC];
                        for (;;) {
#pragma unroll
                            for (int n = 0; n < NV; ++n) {
                                if (head) {
                                    const uint32_t o = src[n] + (uint32_t)min(wide ? lane : lane & 31, ns[n] - 1) * PS;
                                    vm[n] = x2.ld(o + (wide ? 0 : lane >> 5));
                                    vl[n] = vm[n];
                                    if (wide) vl[n] = x2.ld(o + 1);
                                }
#pragma unroll
                                for (int k = 0; k < MC; ++k) {
                                    const int s = sb + k * SG;            // (a load past the splits repeats one)
                                    va[n][k] = x2.ld(src[n] + (uint32_t)(ragged ? min(s, ns[n] - 1) : s < ns[n] ? s : sb) * PS + kP2Stride + col[n]);
                                }
                            }
                            __builtin_amdgcn_sched_barrier(0);
                            uint32_t stale = 0;
#pragma unroll
                            for (int n = 0; n < NV; ++n) {
                                if (head) stale |= (vm[n].y ^ stamp) | (vl[n].y ^ stamp);
#pragma unroll
                                for (int k = 0; k < MC; ++k) stale |= va[n][k].y ^ stamp;
                            }
                            if (stale == 0 || spin.expired(p)) break;
                        }
                        if (head) {
#pragma unroll
                            for (int n = 0; n < NV; ++n) {
                                const float m = __builtin_bit_cast(float, vm[n].x);
                                const float l = wide ? __builtin_bit_cast(float, vl[n].x) : __shfl(m, 32 + (lane & 31));
                                const bool mine = lane < ns[n];           // (up to 32 splits: lanes 32..63 hold sums)
                                const float f = mine ? __builtin_amdgcn_exp2f(m - wave_max(mine ? m : kNegBig)) : 0.f;
                                wgt[n] = f / wave_total(mine ? l * f : 0.f);
                            }
                        }
#pragma unroll
                        for (int n = 0; n < NV; ++n)
#pragma unroll
                            for (int k = 0; k < MC; ++k) {
                                const int s = sb + k * SG;                // (uniform)
                                const float w = lane_of(wgt[n], s & 63);
                                if (s < ns[n]) at[n] = fmaf(__builtin_bit_cast(float, va[n][k].x), w, at[n]);
                            }
                    }
                    if (NV == 1 && SG > 1) {
                        red[sg * cv + v] = at[0];
                    } else {
                        int ex[NV] = {};
                        if constexpr (MF) wave_max_bits(at, ex);
#pragma unroll
                        for (int n = 0; n < NV; ++n) {
                            const int vi = v0 + v + n * NT;
                            if (vi < V) keep(vi, at[n], scale_of(ex[n]));
                        }
                    }
                }
                if (NV == 1 && SG > 1) {
                    lds_barrier();
                    if (tid < cv) {
                        float a = red[tid];
                        for (int k = 1; k < SG; ++k) a += red[k * cv + tid];
                        int ex[1] = {};
                        if constexpr (MF) wave_max_bits({a}, ex);
                        keep(v0 + tid, a, scale_of(ex[0]));
                    }
                }
            }
        };
        using std::integral_constant;
        auto merge = [&](auto ragged_c) {
            constexpr bool ragged = decltype(ragged_c)::value;
            if constexpr (BT > 4) {
                if (V > 2 * NT)
                    run(integral_constant<int, 4>{}, integral_constant<int, 2>{}, ragged_c);
                else if (V > NT)
                    run(integral_constant<int, 2>{}, integral_constant<int, 4>{}, ragged_c);
                else
                    run(integral_constant<int, 1>{}, integral_constant<int, 8>{}, ragged_c);
            } else if (MCW > 4 && (ragged ? row_items[p.B] * HD : p.NS * V) > 4 * NT) {      // more than four splits per thread
                run(integral_constant<int, 1>{}, integral_constant<int, MCW>{}, ragged_c);
            } else {
                run(integral_constant<int, 1>{}, integral_constant<int, 4>{}, ragged_c);
            }
        };
        if (kLayer && row_items)
            merge(integral_constant<bool, kLayer>{});
        else
            merge(integral_constant<bool, false>{});
        // (MFMA tiles: what rows past the batch hold lands in rows of the product nobody reads)
        for (int e = V + tid; !MF && e < BT * HD; e += NT) as[e] = 0.f;
        lds_barrier();
    }
    CF_STAMP(11);           // attention merged

    for (int ch = 0; MF && ch < nchunk; ++ch) {
        const int cbase = c3 * p.CW3 + ch * kOutChunk;
        if (cbase >= p.D) break;
        if (ch > 0) p3_load<HD, MF>(p, lp, tid, hq, c3, rs, ch, tile);
        if constexpr (MF) {
            // [16 batch rows] x [rows of the item] x [128 columns of this wavefront]: one or two steps of 32 rows for each
            // half of the rows, with every part of the attention output
            const int lig = lane & 15, kg = lane >> 4, cb = wv & 3, kh = wv >> 2;
            f32x4 acc4[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) acc4[c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int sstep = 0; sstep < HD / 64; ++sstep) {
                const int row = HD / 2 * kh + 32 * sstep + 8 * kg;      // first of the lane's eight rows
                const h8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
                h8 a[PARTS], f[8];
#pragma unroll
                for (int n = 0; n < PARTS; ++n)
                    a[n] = row < nrows ? *reinterpret_cast<const h8 *>(ap + (n * 16 + lig) * AR + rbeg + row) : zero;
                transpose8(&tile.w[8 * sstep], f);
#pragma unroll
                for (int c = 0; c < 8; ++c)
#pragma unroll
                    for (int n = 0; n < PARTS; ++n) acc4[c] = mfma16(a[n], f[c], acc4[c]);
            }
            // the two halves of the rows -> one partial row per batch row
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float *dst = red + ((kh * 16 + 4 * kg + r) * kOutChunk) + 128 * cb + 8 * lig;
                *reinterpret_cast<f32x4 *>(dst) = f32x4{acc4[0][r], acc4[1][r], acc4[2][r], acc4[3][r]};
                *reinterpret_cast<f32x4 *>(dst + 4) = f32x4{acc4[4][r], acc4[5][r], acc4[6][r], acc4[7][r]};
            }
            lds_barrier();
            static_assert(kOutChunk == NT, "a thread adds one column of every row");
            const float iv = inv[lane & 31];
            const bool mine = cbase + tid < p.D, halves = HD == 128 && nrows > 64;      // (halves: with a factor each)
            for (int b0 = 0; b0 < p.B; b0 += 4) {
                float u[4], v[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    u[k] = red[(b0 + k) * kOutChunk + tid];
                    v[k] = red[(16 + b0 + k) * kOutChunk + tid];          // (rows HD / 2 and on of the item: zero if it has none)
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float f0 = lane_of(iv, 2 * (b0 + k) + rbeg / 64), f1 = lane_of(iv, 2 * (b0 + k) + 1);
                    const float sum = fmaf(u[k], f0, v[k] * (halves ? f1 : f0));
                    if (mine && b0 + k < p.B) x3.st((uint32_t)(slot * p.B + b0 + k) * p.D + cbase + tid, sum, stamp);
                }
            }
            CF_STAMP(18);   // output partial stored
            lds_barrier();
        }
    }
    if constexpr (!MF) {
        float acc[BT][8];
        auto clear = [&]() {
#pragma unroll
            for (int b = 0; b < BT; ++b)
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[b][j] = 0.f;
        };
        // (straight-line code: a branch per row would serialise the LDS reads; a row past the item has a zero tile entry, its
        // is past the end of its buffer, so it may be multiplied by any finite value)
        auto use_row = [&](int u) {
            const int r = rbeg + (lane >> 3) + 8 * min(u, iters - 1);
            float f[8];
            unpack8(tile.w[u], f);
#pragma unroll
            for (int b = 0; b < BT; ++b) {
                const float av = as[b * HD + r];
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[b][j] = fmaf(av, f[j], acc[b][j]);
            }
        };
        // The eight row groups of a wavefront hold the rows of the item, so their sum is the partial: it is folded in
        // registers, a lane ends with one column, and nothing passes through LDS (rows dealt to the wavefronts, whose 512
        // columns were then added through LDS between two barriers, took 0.6 - 1.2 us at batch 1).
        auto publish = [&](int ch) {
            const int cc = c3 * p.CW3 + ch * kOutChunk + 64 * wv + 8 * (lane & 7) + (lane >> 3);
#pragma unroll
            for (int b = 0; b < BT; ++b) {
                float sum[1];
                lanes::fold8<8>(acc[b], sum);
                if (b < p.B && cc < p.D) x3.st((uint32_t)(slot * p.B + b) * p.D + cc, sum[0], stamp);
            }
            CF_STAMP(18);       // output partial stored
        };
        auto use_tile = [&]() {
#pragma unroll
            for (int u = 0; u < OutTile<HD>::MAXR; ++u) {
                use_row(u);
                // (the sums of all batch rows are made here, a few rows of the tile at a time: left alone, the compiler moves those
                // of a batch row to where they are published and keeps the whole tile as fp32 values until the last one)
                if (BT > 1 && u % 4 == 3) {
#pragma unroll
                    for (int b = 0; b < BT; ++b)
#pragma unroll
                        for (int j = 0; j < 8; ++j) asm volatile("" : "+v"(acc[b][j]));
                }
            }
        };
        const int n = min(nchunk, (p.D - c3 * p.CW3 + kOutChunk - 1) / kOutChunk);
        if constexpr (BT == 1) {
            if (n == 1) {
                clear();
                use_tile();
                publish(0);
            } else {
                // Several chunks per item: every register of the tile is requested again, for the next chunk, as soon as it has
                // been used, so that the stream of W_o does not stop between two chunks (the offset depends on the sums the
                // register went into: the request stays behind its last use).  Behind the last chunk there is nothing to load.
                for (int ch = 0; ch < n; ++ch) {
                    const OutRows<HD, false> next(p, lp, tid, hq, c3, rs, ch + 1, ch + 1 < n);
                    clear();
#pragma unroll
                    for (int u = 0; u < OutTile<HD>::MAXR; ++u) {
                        use_row(u);
                        uint32_t off = next.off;
                        asm volatile("" : "+v"(off) : "v"(acc[0][0]), "v"(acc[0][1]), "v"(acc[0][2]), "v"(acc[0][3]), "v"(acc[0][4]),
                                     "v"(acc[0][5]), "v"(acc[0][6]), "v"(acc[0][7]));
                        tile.w[u] = next.row(u, off);
                    }
                    publish(ch);
                }
            }
        } else {
            for (int ch = 0;;) {
                clear();
                use_tile();
                publish(ch);
                if (++ch >= n) break;
                p3_load<HD, MF>(p, lp, tid, hq, c3, rs, ch, tile);
            }
        }
    }
    if constexpr (!MF) lds_barrier();         // the merged values have been read
}

// ---------------------------------------------------------------------------
// Phase 4: every workgroup owns CPW output columns (ceil(D/W), rounded up to an even number) and adds the per-head
// partials of those columns in slot order (the cross-head reduction that the paper
// does with atomicAdd), then writes fp16.
// ---------------------------------------------------------------------------
// The residual input of output value i of this workgroup, which owns the columns [c0, c0 + ncol) (0 when there is none): from x, in a stack past its first layer
// from the slots xin, where this workgroup itself has left it.
__device__ __forceinline__ uint16_t residual_input(const Params &p, int i, int c0, int ncol, float rncol, const uint64_t *xin)
{
    uint16_t r = 0;
    if (kLayer && (p.flags & kFlagResidual) && i < ncol * p.B) {
        const int b = fdiv(i, rncol), c = i - b * ncol;
        const size_t at = (size_t)b * p.D + c0 + c;
        if (xin) {
            const uint32_t two = Xbuf(xin).ld(at >> 1).x;
            r = (uint16_t)(at & 1 ? two >> 16 : two);
        } else {
            r = p.x[at];
        }
    }
    return r;
}

// xout != null (a layer of a stack that is not the last): the result, rounded to fp16 as `out` would hold it, goes to
// the slots the next layer's projection reads its input from, not to `out`.  xin: the slots this layer's input came from.
template <bool FEW, bool STACK, class HookFn>
__device__ __forceinline__ void final_reduce(const Params &p, int tid0, uint32_t stamp, float *smem, uint64_t *xout, const uint64_t *xin, HookFn &&after_polls)
{
    const int tid = tid0;
    const Xbuf x3(p.p3);
    const int nslots = p.nq << p.LRS3;
    const int c0 = blockIdx.x * p.CPW;
    const int ncol = min(p.CPW, p.D - c0);
    const int nv = max(ncol, 0) * p.B;               // values this workgroup produces (none where W * CPW > D)
    const float rncol = reciprocal(ncol);
    int cb, spt, own;
    bool wide;
    uint16_t xres;
    auto fetch = [&](int v0) {                       // the partials of the values v0 .. v0 + cb - 1, added up by slots s0, s0 + spt, ..., to LDS
        cb = min(NT, nv - v0);
        const float rcb = reciprocal(cb);
        spt = min(__builtin_amdgcn_readfirstlane(fdiv(NT, rcb)), nslots);        // slots read in parallel
        const int s0 = fdiv(tid, rcb), v = tid - s0 * cb;
        const int b = fdiv(v0 + v, rncol), c = (v0 + v) - b * ncol;
        // the residual input of the value this thread writes below, on its
        // way while the partials are polled.  (Fetching it before phase 3 was tried: a load inside a branch
        // there makes every later wait for the output-projection tile drain the queue.)
        // Up to 32 values: sixteen lanes add the sums of a value (one thread for up to 256 sums of two values took 0.9 us of
        // the tiny shape, so 0.6); more: one thread each, at most sixteen sums.  (FEW: not in the 16-row kernels, which rarely
        // have so few and lost 1 % to the code.)
        wide = FEW && cb <= NT / 16;
        own = wide ? tid >> 4 : tid;                 // the value whose sums this thread adds
        xres = residual_input(p, v0 + own, c0, ncol, rncol, xin);
        if (s0 < spt) {
            const int n = fdiv(nslots - s0 + spt - 1, reciprocal(spt));
            const uint32_t base = (uint32_t)(s0 * p.B + b) * p.D + c0 + c, stride = (uint32_t)(spt * p.B) * p.D;
            // (more than eight slots per thread: sixteen polls in flight, one round trip instead of two)
            smem[s0 * cb + v] = nslots > 8 * spt ? ll_sum<16>(p, x3, base, stride, n, stamp) : ll_sum<8>(p, x3, base, stride, n, stamp);
        }
        CF_STAMP(19);           // head partials arrived
        lds_barrier();
    };
    auto finish = [&](int v0) {
        float sum = !wide && kLayer && (p.flags & kFlagResidual) ? h2f(xres) : 0.f;
        if (own < cb)
            for (int k = wide ? tid & 15 : 0; k < spt; k += wide ? 16 : 1) sum += smem[k * cb + own];
        if (wide) sum = row_sum<16>(sum);
        if (wide && kLayer && (p.flags & kFlagResidual)) sum = h2f(xres) + sum;
        if (!STACK || !xout) {
            if (own < cb && (!wide || (tid & 15) == 0)) {
                const int bo = fdiv(v0 + own, rncol), co = (v0 + own) - bo * ncol;
                p.out[(size_t)bo * p.D + c0 + co] = f2h(sum);
            }
        } else {
            // pairs of an even value and the one behind it, neighbours of one row (the workgroup's columns are an even number)
            const uint32_t h = f2h(sum);
            float a = __builtin_bit_cast(float, h), n = a;
            if (wide)
                lanes::swap16(a, n);                              // n: the value of the odd row of lanes beside this one
            else
                n = dpp_move<0xF5>(n);                            // quad_perm [1,1,3,3]
            if (own < cb && (own & 1) == 0 && (!wide || (tid & 15) == 0)) {
                const int bo = fdiv(v0 + own, rncol), co = (v0 + own) - bo * ncol;
                Xbuf(xout).st((uint32_t)(bo * p.D + c0 + co) >> 1, __builtin_bit_cast(float, h | __builtin_bit_cast(uint32_t, n) << 16), stamp);
            }
        }
        lds_barrier();
    };
    if (nv > 0) fetch(0);
    after_polls();          // (in one place and in no branch: a stack's next layer counts on what it requests, and the registers that takes hold nothing before)
    if (nv > 0) finish(0);
    for (int v0 = NT; v0 < nv; v0 += NT) {
        fetch(v0);
        finish(v0);
    }
}

// Whether the first half of the output-projection tile is requested before the queries are waited for (the second behind the
// cached rows) and not behind the cached rows (the second behind the stored partial): the memory pipe idles while the q
// partials travel, and the merge finds less of the tile in front of its polls.  Per layer, us: Llama-2-7B shape, 100 / 4096 / 8000
// rows 29.9 / 38.0 / 47.3 -> 28.9 / 37.2 / 46.6, one launch over the layers, 1024 rows 30.6 -> 29.7; D 2056, 14 heads of 64, batch 3
// 20.0 -> 19.2.  With attention on MFMA tiles the registers decide: four heads per group, one or two rows gain at short caches only
// (Llama-3-8B shape, 100 rows 25.0 -> 24.1, 32000 rows 41.7 -> 42.0; a choice at run time costs 1 us, the waits behind it are no
// longer exact), eight heads (37.9 -> 38.8), the 16-row tile (35.2 -> 37.5, spills) and the one-launch stack (25.0 -> 25.4) lose.
template <int HD, int G>
struct EarlyTile {
    static constexpr bool on = !AttnMfma<HD, G>::on;
};

// Splits that the merge of phase 3 has in flight where a thread adds more than four (the sums and their order are the same).
// Four in the one-launch stack with one batch row and up to two query heads per KV head: the next layer's weights fill the
// registers there, and eight made the kernel spill 20 bytes per lane.
template <int HD, int G, int BT, bool STACK>
struct MergeWide {
    static constexpr int n = STACK && BT == 1 && G <= 2 ? 4 : 8;
};

// LDS floats of phases 2 and 3: the same expressions as in lds_floats, where the host adds the table of the rows' first items.
constexpr size_t p2_lds_floats(int hd, int g)
{
    const bool ma = hd == 128 && g >= 4;                                          // attention on MFMA tiles: a K tile per wavefront
    return (size_t)hd + (size_t)(g + 2) * hd + 8 + 2 * (size_t)g * kWaves + (size_t)g * kWaves * hd +          // partials folded through LDS
           (ma ? (size_t)kWaves * 32 * (hd + 8) / 2 + 2 * 256 * 4 : 0);           // K tiles, q operands
}
// merged attention rows, then the sums of the merge (one per thread) or, on MFMA tiles, the two halves of the product
constexpr size_t p3_lds_floats(int hd, int bt)
{
    return mfma_tiles(bt) ? (size_t)out_operand_floats(hd) + (size_t)2 * bt * kOutChunk : (size_t)bt * hd + kThreads;
}
template <int HD, int G, int BT>
constexpr size_t kRowTable = p2_lds_floats(HD, G) > p3_lds_floats(HD, BT) ? p2_lds_floats(HD, G) : p3_lds_floats(HD, BT);

// The kernel's arguments, through a pointer the compiler cannot connect with an earlier one (see decode_steps).
//
// At small shapes the time between two hand-overs is the time to issue the instructions in between (one every four to eight
// clocks and wavefront; 1300 a wavefront at the tiny shape, half of them scalar).  Us a layer, before / after: the arguments by
// phase, loads that end with their buffer, divisions by reciprocals, no copies of loaded registers where paths meet:
// tiny shape 13.7 / 11.6, D 2056, 14 heads of 64, batch 3 19.4 / 16.3, 1024 columns, 8 heads of 128, batch 1 15.4 / 12.9,
// 16 heads of 64 over 8, batch 5, norm 26.3 / 21.4, Llama-3-8B shape, norm, 1000 rows, batch 1 / 16 26.8 / 24.0 and 46.8 / 42.7,
// one launch, norm, 2048 rows 24.9 / 23.5, Llama-2-7B shape 36.4 / 35.1, Llama-2-70B shape 75.1 / 73.4 (of which 0.5 the stream of W_o).
__device__ __forceinline__ const Params &kernarg_params()
{
    typedef const __attribute__((address_space(4))) Params *KernargParams;
    KernargParams pk = (KernargParams)__builtin_amdgcn_kernarg_segment_ptr();      // (StackArgs begins with Params)
    asm volatile("" : "+s"(pk));
    return *(const Params *)pk;
}

// One launch = n_layers decode steps in a row (1 for the plain entry points).  Layer l > 0 takes its weights and
// caches from tab[l] and its input from the slots xslots, where the final reduction of layer l - 1 left its result;
// the last layer writes `out`.  Nothing separates the layers but those slots: a workgroup goes on as soon as the
// rows of the input it needs have arrived.  The exchange areas need no second set: a workgroup can post values of
// layer l + 1 only after it has taken in that layer's input, which exists only when every workgroup has finished
// reading what layer l exchanged.
template <int HD, int G, int BT, bool STACK>
__device__ __forceinline__ void decode_steps(const Params &p0, const LayerPtrs *tab, int n_layers_in, uint64_t *xslots)
{
    const int n_layers = STACK ? n_layers_in : 1;
    extern __shared__ __align__(16) float smem[];
    {
        // The compiler loads each kernel argument shortly before its first use: several dependent
        // round trips to cold memory in a row at the start of every launch.  One word of every 64-byte
        // line of the argument block is read here, all at once, so the later reads hit the scalar cache.
        static_assert(sizeof(Params) == 320, "one load per 64-byte line of the argument block below");
        auto ka = __builtin_amdgcn_kernarg_segment_ptr();
        uint32_t t0, t1, t2, t3, t4;
        asm volatile("s_load_dword %0, %5, 0x0\n\ts_load_dword %1, %5, 0x40\n\ts_load_dword %2, %5, 0x80\n\t"
                     "s_load_dword %3, %5, 0xc0\n\ts_load_dword %4, %5, 0x100\n\ts_waitcnt lgkmcnt(0)"
                     : "=&s"(t0), "=&s"(t1), "=&s"(t2), "=&s"(t3), "=&s"(t4)
                     : "s"(ka));
    }
    __shared__ float s_rope[RopeRows<HD, BT>::ROWS * HD];    // cos / sin of the RoPE angles, per row if the rows differ
    const int tid = threadIdx.x;
    // Workgroup w runs on die (XCD) w % 8, and the odd dies get about a tenth less memory
    // bandwidth than the even ones.  With pairmap a team sits on one pair of dies, members with an
    // even index on the even die: those take the longer splits of the cached rows.
#if CF_STAMPS
    if (tid < kStamps) s_ts[tid] = 0;       // same wavefront as thread 0: ordered before its stamps
#endif
    CF_STAMP(0);
#if CF_STAMPS
    if (tid == 0)   // where this workgroup runs: XCC id and the HW_ID register (CU, SE ...)
        s_ts[7] = ((unsigned long long)__builtin_amdgcn_s_getreg(63508) << 32) | (unsigned)__builtin_amdgcn_s_getreg(63492);
#endif

    unsigned long long cnt0 = 0;
    P1Regs<HD, BT> rg;
    bool primed = false;
    if (STACK) {
        // the RoPE table is the same for all layers (one position; a stack has no per-row positions): built here,
        // outside the loop, so that its fp64 constants do not become loop-invariant registers
        for (int e = tid; e < HD / 2; e += NT)
            rope_cos_sin(p0.pos, rope_inv_freq(e, HD, p0.rope_log2_base), s_rope[e], s_rope[HD / 2 + e]);
        lds_barrier();
    }
    for (int layer = 0; layer < n_layers; ++layer) {
    // In a stack the parameters are read through a pointer to the kernel's argument block that is made opaque per
    // layer (as are the thread and workgroup index below): whatever depends only on them is loop-invariant, and
    // the compiler would otherwise compute all of it once in front of the loop over the layers and keep it in
    // registers, hundreds of values, across every phase.
    // The same at the start of every phase: what a phase takes from the arguments, it fetches itself (hits in the scalar cache)
    // and does not keep beyond its end.  With one reference for all phases more scalars were alive than there are registers,
    // and every one moved to a vector register's lane and back is an instruction each way, hundreds of them.
    const Params &p = kernarg_params();
    int n2 = p.B * p.NS;                             // attention items of the team
    const int n3 = G * (p.NC3 << p.LRS3);            // output-projection items of the team
    // (in a stack the thread index is made opaque per layer: everything derived from it would otherwise be computed
    // once in front of the loop over the layers and be kept in registers across all phases)
    int tl = threadIdx.x, w = blockIdx.x;
    if (STACK) asm volatile("" : "+v"(tl), "+s"(w));
    const int team_round = qdiv(w >> p.pairmap, p.div_nkv);
    const int team = (w >> p.pairmap) - team_round * p.nkv, member = (team_round << p.pairmap) | (w & p.pairmap);
    // weights and caches of this layer (layer 0, and the only layer of a plain call: those of the parameters);
    // a reference into the argument block either way, so that each pointer is fetched where it is used
    static_assert(offsetof(Params, wo) == offsetof(Params, wqkv) + 8 && offsetof(Params, kc) == offsetof(Params, wqkv) + 16 &&
                      offsetof(Params, vc) == offsetof(Params, wqkv) + 24 && offsetof(Params, gamma) == offsetof(Params, wqkv) + 32,
                  "Params holds a LayerPtrs");
    const LayerPtrs &lp = (STACK && layer > 0) ? tab[layer] : *reinterpret_cast<const LayerPtrs *>(&p.wqkv);
    KvBuf<HD, G> kv;
    OutTile<HD> tile;
    // the first attention item.  With positions per row the stream is set up only where phase 1 first needs it: the positions come from
    // memory, and waiting for them here would hold up the first weight loads.
    const bool own_pos = kLayer && p.row_pos != nullptr;
    int lens = 0;
    RowItem ri;
    ri.b = member < n2 ? qdiv(member, p.div_ns) : 0;
    ri.s = member < n2 ? member - ri.b * p.NS : 0;
    ri.ns = p.NS;
    ri.first = ri.b * p.NS;
    const int pos_first = row_pos(p, ri.b);
    P2Stream<HD, G> st2 = P2Stream<HD, G>::planned(p, lp, tl, team, ri.b, ri.s, own_pos ? 0 : p.pos, member < n2 && !own_pos);

    // ---- phase 1 (projection); its last step already starts the K/V stream of phase 2
    EarlyQ<STACK ? 8 : 16> eq;
    // (without batches requested ahead the registers of the two batches belong to this layer alone)
    P1Regs<HD, BT> rg_layer;
    P1Regs<HD, BT> &rgu = (STACK && P1Ahead<HD, G, BT>::n > 0) ? rg : rg_layer;
    const uint32_t stamp = p1_all<HD, G, BT, STACK, 0>(p, lp, tl, team, member, smem, s_rope, STACK ? layer : 0, xslots, n_layers, cnt0,
                                             rgu, primed, lens, [&](int stage) {
                                                 // (here, where two batches of weights are in flight: in front of the first one it
                                                 // delayed the second, 0.8 us with 16 rows)
                                                 if (kLayer && !STACK && p.ragged)
                                                     ri = deal_rows<HD>(p, tl & 63, (tl & 15) < p.B ? min(max(lens, 0), p.pos) : 0, member, ri);
                                                 if (kLayer && !STACK && ri.items)
                                                     st2 = P2Stream<HD, G>(p, lp, tl, team, ri.b, ri.t0, ri.t1, ri.pos);
                                                 else if (own_pos)
                                                     st2 = P2Stream<HD, G>::planned(p, lp, tl, team, ri.b, ri.s, pos_first, member < n2);
                                                 st2.prefetch(kv, 0);
                                             });
    const bool ragged = kLayer && !STACK && ri.items != 0;
    if (ragged) n2 = ri.items;
    // first items of the rows for the merge of phase 3, behind what the phases up to there hold in LDS (phase 1 is over in this
    // workgroup: whoever took part in it has passed its last barrier)
    int *row_items = reinterpret_cast<int *>(smem + kRowTable<HD, G, BT>);
    if (ragged && tl <= kMaxRows) row_items[tl] = ri.table;
    // a first look at the team's q partials (in a stack only for one batch row and attention on the vector ALU: no
    // registers are left for the sixteen pairs there, they would be spilled as they arrive)
    if (member < n2 && !(STACK && (AttnMfma<HD, G>::on || BT > 1)))
        eq.template issue<HD, G>(p, tl, team, ri.b, NewTokenFirst<HD, G, BT>::selectors(ri.s == ri.ns - 1));
    st2.prefetch(kv, 1);
    CF_STAMP(1);
    // ---- phase 2 (attention); the last item already starts the W_o stream of phase 3
    auto p3_args = [&](const Params &q, int it, int &hq, int &c3, int &rs) {
        const int g = qdiv(it, q.div_n3), rem = it - g * (q.NC3 << q.LRS3);
        hq = team * G + g;
        c3 = rem >> q.LRS3;
        rs = rem & ((1 << q.LRS3) - 1);
    };
    auto layer_ptrs = [&](const Params &q) -> const LayerPtrs & {
        return (STACK && layer > 0) ? tab[layer] : *reinterpret_cast<const LayerPtrs *>(&q.wqkv);
    };
    constexpr bool EARLY = EarlyTile<HD, G>::on;
    if (EARLY) {
        // (no branch around the loads, an empty buffer instead: the waits for the cached rows count them)
        const Params &q = kernarg_params();
        int hq, c3, rs;
        p3_args(q, member < n3 ? member : 0, hq, c3, rs);
        p3_load<HD, Mfma<HD, BT>::on>(q, layer_ptrs(q), tl, hq, c3, rs, 0, tile, 0, member < n2 && member < n3);
    }
    auto p3_prefetch = [&](int part) {
        if (member < n3) {
            const Params &q = kernarg_params();
            int hq, c3, rs;
            p3_args(q, member, hq, c3, rs);
            p3_load<HD, Mfma<HD, BT>::on>(q, layer_ptrs(q), tl, hq, c3, rs, 0, tile, part);
        }
    };
    if (member < n2) {
        for (int it = member;;) {
            const Params &q = kernarg_params();
            const int next = it + q.TS;
            const bool more_items = next < n2;
            // stage 1: first half of the output-projection tile, stage 2: second half (early: stage 1 the second half)
            p2_item<HD, G, BT>(q, layer_ptrs(q), tl, team, ri.b, ri.s, ri.ns, ri.first, stamp, it == member, st2, kv, eq, smem,
                               s_rope + (kLayer && q.row_pos ? ri.b * HD : 0), [&](int stage) {
                if (!more_items && (!EARLY || stage == 1)) p3_prefetch(EARLY ? 1 : stage - 1);
            });
            if (!more_items) break;
            it = next;
            const Params &qn = kernarg_params();
            ri.b = qdiv(it, qn.div_ns);
            ri.first = ri.b * qn.NS;
            ri.s = it - ri.first;
            st2 = P2Stream<HD, G>::planned(qn, layer_ptrs(qn), tl, team, ri.b, ri.s, row_pos(qn, ri.b));
            st2.prefetch(kv, 0);
            st2.prefetch(kv, 1);
        }
    } else {
        p3_prefetch(2);
    }
    CF_STAMP(3);
    const bool more = STACK && layer + 1 < n_layers;
    auto no_next = [](int) {};
    const LayerPtrs &lpn = STACK ? tab[more ? layer + 1 : layer] : lp;
    constexpr int AHEAD = STACK ? P1Ahead<HD, G, BT>::n : 0;
    // ---- phase 3 (output projection, per-head partials)
    // (The tile of the first item is on its way, that of a further one is requested when the item before is done.  A load in front
    // of the merge for the items that need it is a second source of the tile's registers there: they were copied, and the copy
    // waited for the whole tile before the first poll went out.)
    if (ragged) lds_barrier();               // (a member without an attention item has passed no barrier since its table)
    if (member < n3) {
        for (int it = member;;) {
            const Params &q = kernarg_params();
            int hq, c3, rs;
            p3_args(q, it, hq, c3, rs);
            p3_item<HD, BT, MergeWide<HD, G, BT, STACK>::n>(q, layer_ptrs(q), tl, hq, c3, rs, stamp, tile, smem, ragged ? row_items : nullptr);
            it += q.TS;
            if (it >= n3) break;
            const Params &qn = kernarg_params();
            p3_args(qn, it, hq, c3, rs);
            p3_load<HD, Mfma<HD, BT>::on>(qn, layer_ptrs(qn), tl, hq, c3, rs, 0, tile);
        }
    }
    CF_STAMP(4);
    // ---- phase 4 (sum over heads)
    // In a stack the first two batches of the next layer's weights are requested here: one before the partial
    // outputs of the heads are waited for, one once they have arrived (behind both, their polls would queue for
    // the time the batches take to stream in).
    // (measured on the 7B shape, us per layer: this placement 36.5; both batches before the wait 37.6; the first
    // one already after the merge of the attention partials 37.7; none 37.6)
    if (AHEAD >= 1)
        p1_all<HD, G, BT, STACK, 1>(kernarg_params(), lpn, tl, team, member, smem, s_rope, 0, nullptr, n_layers, cnt0, rg, more, lens, no_next);
    final_reduce<(BT <= 4), STACK>(kernarg_params(), tl, stamp, smem, more ? xslots : nullptr, layer > 0 ? xslots : nullptr, [&]() {
        if (AHEAD >= 2)
            p1_all<HD, G, BT, STACK, 2>(kernarg_params(), lpn, tl, team, member, smem, s_rope, 0, nullptr, n_layers, cnt0, rg, more, lens, no_next);
    });
    primed = more;
    CF_STAMP(5);
    }   // layers
    if (tid == 0) p0.done[(size_t)blockIdx.x * kCounterStride] = cnt0 + (unsigned long long)(n_layers - 1);   // steps completed
#if CF_STAMPS
    CF_STAMP(6);
    lds_barrier();
    if (p0.dbg_t && tid < kStamps) p0.dbg_t[(size_t)blockIdx.x * kStamps + tid] = s_ts[tid];
#endif
}

template <int HD, int G, int BT>
__global__ void __launch_bounds__(NT) CF_KERNEL(const Params p)
{
    decode_steps<HD, G, BT, false>(p, nullptr, 1, nullptr);
}

// A stack of layers in one launch: the argument block carries the table of per-layer pointers by value.
#if CF_LAYER
#define CF_STACK_KERNEL fused_layer_stack
#else
#define CF_STACK_KERNEL fused_decode_stack
#endif
template <int HD, int G, int BT>
__global__ void __launch_bounds__(NT) CF_STACK_KERNEL(const StackArgs a)
{
    decode_steps<HD, G, BT, true>(a.p, a.tab, a.n_layers, a.xslots);
}

#if !CF_LAYER
// One-time rearrangement of the weights into per-head contiguous blocks (16 bytes per thread step).
__global__ void pack_qkv_kernel(const uint4 *__restrict__ src, uint4 *__restrict__ dst, int D, int nqkv, int hd)
{
    const size_t n = (size_t)D * nqkv / 8;
    const int v_per_row = hd / 8;
    const size_t blk = (size_t)v_per_row * D + kQkvBlockPad / 16;      // block stride in 16-byte units
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const size_t c8 = i % v_per_row, r = (i / v_per_row) % D, cb = i / ((size_t)v_per_row * D);
        dst[cb * blk + r * v_per_row + c8] = src[(r * nqkv + cb * hd) / 8 + c8];
        if (r == 0 && c8 == 0)
            for (int k = 0; k < kQkvBlockPad / 16; ++k) dst[cb * blk + (size_t)v_per_row * D + k] = make_uint4(0, 0, 0, 0);
    }
}

__global__ void pack_o_kernel(const uint4 *__restrict__ src, uint4 *__restrict__ dst, int D, int nq, int hd)
{
    const int nch = (D + kOutChunk - 1) / kOutChunk;
    const size_t n = (size_t)nq * nch * hd * (kOutChunk / 8);
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const size_t c8 = i % (kOutChunk / 8), r = (i / (kOutChunk / 8)) % hd;
        const size_t ch = (i / ((size_t)(kOutChunk / 8) * hd)) % nch, h = i / ((size_t)(kOutChunk / 8) * hd * nch);
        const size_t col = ch * kOutChunk + c8 * 8;
        dst[i] = col < (size_t)D ? src[((h * hd + r) * D + col) / 8] : make_uint4(0, 0, 0, 0);
    }
}

#endif  // !CF_LAYER

using KernelFn = void (*)(const Params);

template <int HD, int G>
KernelFn pick_bt(int bt)
{
    switch (bt) {
    case 1: return CF_KERNEL<HD, G, 1>;
    case 4: return CF_KERNEL<HD, G, 4>;
    case 16: return CF_KERNEL<HD, G, 16>;
    default: return nullptr;
    }
}

template <int HD>
KernelFn pick_g(int g, int bt)
{
    switch (g) {
    case 1: return pick_bt<HD, 1>(bt);
    case 2: return pick_bt<HD, 2>(bt);
    case 4: return pick_bt<HD, 4>(bt);
    case 8: return pick_bt<HD, 8>(bt);
    default: return nullptr;
    }
}

KernelFn pick(int hd, int g, int bt)
{
    if (hd == 64) return pick_g<64>(g, bt);
    if (hd == 128) return pick_g<128>(g, bt);
    return nullptr;
}

using StackFn = void (*)(const StackArgs);

template <int G>
StackFn pick_stack_bt(int bt)
{
    if (bt == 1) return CF_STACK_KERNEL<128, G, 1>;
#if !CF_LAYER                                           // (with norm or residual: batch 1 only)
    if (bt == 4) return CF_STACK_KERNEL<128, G, 4>;
    if (bt == 16) return CF_STACK_KERNEL<128, G, 16>;
#endif
    return nullptr;
}

// (head_dim 128 only: the shapes whose stacks are worth one launch)
StackFn pick_stack(int hd, int g, int bt)
{
    if (hd != 128) return nullptr;
    switch (g) {
    case 1: return pick_stack_bt<1>(bt);
    case 2: return pick_stack_bt<2>(bt);
    case 4: return pick_stack_bt<4>(bt);
    case 8: return pick_stack_bt<8>(bt);
    default: return nullptr;
    }
}

}  // namespace

static hipError_t occupancy_of(KernelFn fn, size_t lds_bytes, int *out)
{
    *out = 0;
    if (!fn) return hipSuccess;
    if (lds_bytes > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) return e;
    }
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(out, reinterpret_cast<const void *>(fn), kThreads, lds_bytes);
}

static hipError_t launch_of(KernelFn fn, const Params &p, size_t lds_bytes, hipStream_t stream)
{
    if (!fn) return hipErrorInvalidDeviceFunction;
    hipLaunchKernelGGL(fn, dim3(p.W), dim3(kThreads), lds_bytes, stream, p);
    return hipGetLastError();
}

static hipError_t launch_stack_of(StackFn fn, const StackArgs &a, size_t lds_bytes, hipStream_t stream)
{
    if (!fn || a.p.row_pos || a.n_layers < 1 || a.n_layers > kMaxStackLayers) return hipErrorInvalidDeviceFunction;
    // all workgroups must be resident, as for the one-layer kernel
    int per_cu = 0;
    if (lds_bytes > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) return e;
    }
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(fn), kThreads, lds_bytes);
    if (e != hipSuccess) return e;
    int dev = 0, cus = 0;
    if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
    if ((long)per_cu * cus < a.p.W) return hipErrorLaunchOutOfResources;
    hipLaunchKernelGGL(fn, dim3(a.p.W), dim3(kThreads), lds_bytes, stream, a);
    return hipGetLastError();
}

#if CF_LAYER

hipError_t launch_layer_stack(const StackArgs &a, int hd, int g, int bt, size_t lds_bytes, hipStream_t stream)
{
    return launch_stack_of(pick_stack(hd, g, bt), a, lds_bytes, stream);
}

hipError_t max_workgroups_per_cu_layer(int hd, int g, int bt, size_t lds_bytes, int *out)
{
    return occupancy_of(pick(hd, g, bt), lds_bytes, out);
}

hipError_t launch_fused_layer(const Params &p, int hd, int g, int bt, size_t lds_bytes, hipStream_t stream)
{
    return launch_of(pick(hd, g, bt), p, lds_bytes, stream);
}

#else

bool wants_layer_kernel(const Params &p)
{
    return p.gamma != nullptr || (p.flags & kFlagResidual) != 0 || p.row_pos != nullptr;
}

size_t lds_floats(const Params &p, int hd, int g, int bt)
{
    const size_t maxi = bt == 1 ? 4 : (bt <= 4 ? 2 : 1);
    const size_t f1 = x_lds_floats(hd, bt, p.RPS, wants_layer_kernel(p)) + maxi * kWaves * bt * hd + (size_t)kWaves * bt;
    const size_t table = p.ragged ? kMaxRows + 1 : 0;
    const size_t f2 = p2_lds_floats(hd, g) + table, f3 = p3_lds_floats(hd, bt) + table;
    size_t f = f1 > f2 ? f1 : f2;
    return f > f3 ? f : f3;
}

hipError_t max_workgroups_per_cu(int hd, int g, int bt, size_t lds_bytes, bool layer, int *out)
{
    if (layer) return max_workgroups_per_cu_layer(hd, g, bt, lds_bytes, out);
    return occupancy_of(pick(hd, g, bt), lds_bytes, out);
}

hipError_t launch_pack(const uint16_t *wqkv, const uint16_t *wo, uint16_t *wqkv_p, uint16_t *wo_p, int D, int nqkv,
                       int nq, int hd, hipStream_t stream)
{
    hipLaunchKernelGGL(pack_qkv_kernel, dim3(2048), dim3(256), 0, stream, reinterpret_cast<const uint4 *>(wqkv),
                       reinterpret_cast<uint4 *>(wqkv_p), D, nqkv, hd);
    hipLaunchKernelGGL(pack_o_kernel, dim3(2048), dim3(256), 0, stream, reinterpret_cast<const uint4 *>(wo),
                       reinterpret_cast<uint4 *>(wo_p), D, nq, hd);
    return hipGetLastError();
}

hipError_t launch_fused_stack(const StackArgs &a, int hd, int g, int bt, size_t lds_bytes, hipStream_t stream)
{
    if (wants_layer_kernel(a.p)) return launch_layer_stack(a, hd, g, bt, lds_bytes, stream);
    return launch_stack_of(pick_stack(hd, g, bt), a, lds_bytes, stream);
}

hipError_t launch_fused(const Params &p, int hd, int g, int bt, size_t lds_bytes, hipStream_t stream)
{
    if (wants_layer_kernel(p)) return launch_fused_layer(p, hd, g, bt, lds_bytes, stream);
    return launch_of(pick(hd, g, bt), p, lds_bytes, stream);
}

#endif  // CF_LAYER

}  // namespace cf
