// Fused decode step of a weight-absorbed Multi-Head Latent Attention block (paper Appendix B, Alg. 4) as ONE
// kernel for gfx950, behind the C ABI (cf_mla_* in include/cfdecode.h).
//
// Alg. 4 runs one cluster per head and moves data between its blocks with three ClusterGathers and three
// ClusterReduces.  This kernel (batch 2 to 16; batch 1: cf_mla_heads.hip) has 16 co-resident workgroups per head and
// five hand-overs through global memory; all products run on MFMA tiles with the batch (or the heads) as the 16-row edge:
//
//   A  projections        [q | kv_new] = x [W_Q | W_KV]           64 columns x up to 4 row slices per workgroup
//   B  up-projection      q_lat_i = q_nope_i W_Up[i]              (head i, member j): 1/16 of the kv_lora_rank columns, and
//                         two of the rotary pairs of q_i
//   C  attention          unit of work = (batch row, token range, group of heads), NOT the head: all heads share every
//                         cached row (one latent "head": MQA), so the scores and the weighted sums of the heads against
//                         a tile of 64 rows are two dense products; a row is read from HBM once for all heads.  The
//                         first range also appends the new row and counts the new token
//   D  merge              (head i, member j): 1/16 of the latent dimensions over the ranges (Alg. 4's online-softmax
//                         reduction)
//   E1 down- and output   every member: a_i = z_i W_Down[i], redundantly (131 KB, from the die's L2, for one hand-over
//      projection         less), then rows of W_O of head i, 1/16 of the output columns: a partial of out per head
//   E2 sum over heads     every workgroup: 1/W of the output columns (the paper's atomicAdd)
//
// Two kinds of hand-over.  The last one, few values per reader, goes through stamped {value, stamp} slots
// (cf_team_device.h): one trip.  The others move 32 - 64 KB per reader, where 8 bytes per value and polling every one of
// them is what takes the time (74 KB of query slots took 8 us): the values are written as they are, 4 bytes each, with
// write-through stores; a workgroup waits until its stores have been acknowledged, then writes one flag word, the
// stamp of the launch; a reader polls the flags of its sources and fetches the values with 16-byte loads that, like the
// polls, do not look into its caches.
//
// Measured (DeepSeek-V2-Lite shape, 4096 rows): 16 batch rows 63.8 -> 44.8 us, batch 2 / 4 / 8 36.6 / 44.1 / 52.6 ->
// 32.4 / 33.5 / 37.4, against the kernel that sent everything through slots.  Time line at 16 rows, us from kernel
// start, mean / latest workgroup, launches back to back: A posted 4.5 / 7.0, up-projection 9.2, B posted 9.7 / 10.6, sources there 13.4 / 14.4,
// query operands built 14.9, rows consumed 25.5 / 27.3 (7 TB/s), range posted 28.1 / 30.0, its sources there 32.2 / 33.4, z posted
// 34.2 / 35.8, a_i 38.8 / 39.9, partial of out 40.3, end 42.8 / 43.4.  What bounds it is the chain of stages and hand-overs: behind B and C 3.7
// and 4.1 us from the mean post to the mean arrival, 2.8 and 2.2 from the latest post.
// Each stage requests its weights (or cached rows) before it waits for its input.  All waits are bounded
// (CF_ETIMEOUT), all workgroups have to be resident at once.
#include "cf_lanes_device.h"
#include "cf_mfma_device.h"
#include "cf_mla_internal.h"
#include "cf_plan_arith.h"
#include "cf_rope_device.h"
#include "cf_team_device.h"

#include <cmath>
#include <cstring>
#include <new>

namespace {

using cf::team::Exchange;
using cf::team::pair_t;
constexpr int NT = 512;             // threads per workgroup
constexpr int NW = NT / 64;
constexpr int TS = 16;              // workgroups per head (team)
constexpr int L = 512;              // kv_lora_rank the lane mapping is written for
constexpr int R = 64;               // rope_dim
constexpr int LR = L + R;
constexpr int LJ = L / TS;          // latent dimensions per member: 32
constexpr int HT = 16;              // heads (batch rows) of one MFMA tile: the most the kernel takes
constexpr int MAXBATCH = 16;
constexpr int kMaxSlices = 4;       // row slices of the projections
constexpr int kCounterStride = 16;
constexpr int kTile = 64;           // cached rows per attention tile of a workgroup (held in LDS)
constexpr int KSTR = LR + 8;        // row stride (fp16 values) of the tile in LDS
constexpr int kSteps = LR / 32;     // MFMA steps of a score product (contraction over 576 dimensions)
constexpr int kQops = kSteps * 64;  // 16-byte query operands (one per step and lane)
constexpr int SSTR = kTile + 4;     // row stride (floats) of the scores in LDS
constexpr int AS = 132;             // row stride (floats) of a_i in LDS
constexpr int kMaxSplits = 32;      // token ranges per batch row at most
// LDS, floats.  A: [NW][16][64]; B: [4][16][LJ]; C: query operands, new row, scores, maxima / sums, tile (later the second
// half's accumulators); E1: a_i, [NW][16][128]; E2: [4][128]
constexpr int kLdsC = 2 * kQops * 4 + LR + NW * HT + 2 * HT * SSTR + 4 * HT, kLdsTile = kTile * KSTR / 2;
constexpr size_t kLdsFloats = kLdsC + (kLdsTile > HT * L ? kLdsTile : HT * L);
static_assert(kLdsFloats >= 16 * AS + NW * 16 * 128 && kLdsFloats * 4 <= 160 * 1024, "largest stage");
constexpr float kNegBig = -1.0e30f;
constexpr int kHeadsBatch = 1;      // up to this batch cf_mla_decode runs the head-team kernel (measured cross-over)

using cf::mfma::f32x4;
using cf::mfma::h8;
using cf::mfma::mfma16;
using cf::mfma::transpose8;
using cf::mfma::u32x4;

struct MlaArgs {
    const uint16_t *x, *wq, *wkv, *wup, *wdown, *wo;
    uint16_t *cache, *out;
    uint64_t *slots;                // stamped slots of the last hand-over: [nh][B][D]
    float *data;                    // the other hand-overs' values, 4 bytes each
    uint32_t *flags;                // their flags: [4][256]
    unsigned long long *counters;
    uint32_t *err;
    size_t x1, xq, x3, xml, xz;     // first value of each exchange area: [ksa][B][CQ], [B][nh][LR], [item][HT][L],
                                    // [item][HT][2], [B][nh][L]
    int D, nh, n, v, B, pos, max_seq, W;
    int NS, tps, HG;                // token ranges per batch row, cached rows per range, heads per attention item
    int ksa, rows;                  // row slices of the projections, rows per slice
    float scale_log2e;              // log2(e) / sqrt(nope_dim + rope_dim)
    double log2_base;
    long long spin_ticks;
};

__device__ __forceinline__ uint16_t f2h(float f) { return __builtin_bit_cast(uint16_t, (_Float16)f); }

// Exchanged values without stamps: write-through stores, loads that bypass the caches (agent scope, as put / peek).
struct Data {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ explicit Data(const float *base)
        : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, 0xfffffff0u, 0x00020000)) {}
    __device__ __forceinline__ float ld1(size_t i) const { return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (unsigned)(i * 4), 0, 16)); }
    __device__ __forceinline__ f32x4 ld4(size_t i) const { return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (unsigned)(i * 4), 0, 16)); }
    __device__ __forceinline__ void st1(size_t i, float v) const { __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, (unsigned)(i * 4), 0, 16); }
    __device__ __forceinline__ void st4(size_t i, const f32x4 &v) const { __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, (unsigned)(i * 4), 0, 16); }
};

// Workgroup barrier that orders LDS accesses only.  __syncthreads() would also wait for every outstanding global
// access of the wavefront (vmcnt(0)).  Nothing here passes data between the threads of a workgroup through global memory.
__device__ __forceinline__ void lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// All threads: once every store of the workgroup has been acknowledged (a store counts in vmcnt until then, and a
// write-through store is acknowledged by the memory side), the flag says so.
__device__ __forceinline__ void post(uint32_t *flag, uint32_t stamp)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_sync();
    asm volatile("" ::: "memory");
    if (threadIdx.x == 0) __hip_atomic_store(flag, stamp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Waits for one flag (threads with nothing to wait for pass `on` = false).
__device__ __forceinline__ void wait_flag(const Exchange &x, const uint32_t *flag, bool on)
{
    long long t0 = 0;
    while (on && __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != x.stamp)
        if (cf::team::gave_up(x, t0)) break;
    asm volatile("" ::: "memory");              // what the flag announces is fetched behind it
}

// v = hi + lo with both parts fp16, for the query of the cached rows' scores: 22 bits of values around one, an absolute step
// of 2^-24 below, no more than 65504.
__device__ __forceinline__ void split_hi_lo(const float (&v)[8], h8 &hi, h8 &lo)
{
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        hi[k] = (_Float16)v[k];
        lo[k] = (_Float16)(v[k] - (float)hi[k]);
    }
}

// Three fp16 parts of a scaled row (cf_mfma_device.h) cost 0.65 us of a step (batch 2 / 4 / 16: 32.4 / 33.5 / 44.6 us with
// unscaled pairs, 33.1 / 34.1 / 45.25 us); rounded parts, each with its conversion back, and a scale taken out of every
// accumulator cost 1.45 us.
using cf::mfma::Split;
using cf::mfma::max_abs;
using cf::mfma::row_max;
using cf::mfma::scale_exp;
using cf::mfma::split_scaled;

__device__ __forceinline__ float ror8_add(float v)     // v + the value of the lane 8 further in the row of 16 lanes
{
    return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x128, 0xF, 0xF, true));
}

// Dimension of a cached row that contraction slot (step m, lane group g, element 0) of a score product stands for:
// a lane reads 32 contiguous bytes of the row in two steps, the four groups of a token one 128-byte line.
__device__ __forceinline__ int score_dim(int m, int g) { return 64 * (m >> 1) + 16 * g + 8 * (m & 1); }

// Stage time stamps of every workgroup, only in builds with -DCF_STAMPS=1 (the profiling library).
#ifndef CF_STAMPS
#define CF_STAMPS 0
#endif
#if CF_STAMPS
constexpr int kMlaStamps = 16;
__device__ unsigned long long g_mla_ts[256 * kMlaStamps];
#define MLA_STAMP(k) do { if (threadIdx.x == 0) s_ts[k] = wall_clock64(); } while (0)
#else
#define MLA_STAMP(k)
#endif

__global__ void __launch_bounds__(NT) fused_mla_decode(const MlaArgs a)
{
    extern __shared__ __align__(16) float smem[];                    // carved anew by every stage
    __shared__ float s_rope[R];                         // cos, sin of the rotary angles
    __shared__ __align__(16) float s_f[16 * NW];        // 1 / scale of operand row (batch row) and wavefront
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, w = blockIdx.x;
    // workgroup w runs on die w % 8; with a multiple of eight heads a head's members share one die and its L2
    const int head = a.nh % 8 == 0 ? w % 8 + 8 * (w / 8 / TS) : w / TS, j = a.nh % 8 == 0 ? w / 8 % TS : w % TS;
    const int B = a.B, nr = a.n + R, CQq = a.nh * nr, CQ = CQq + LR;
    const int g = lane >> 4, c = lane & 15;                            // contraction group, operand row / column of the lane
    const h8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
    uint32_t *fA = a.flags, *fB = a.flags + 256, *fC = a.flags + 512, *fD = a.flags + 768;
#if CF_STAMPS
    __shared__ unsigned long long s_ts[kMlaStamps];
    if (tid < kMlaStamps) s_ts[tid] = 0;
#endif
    MLA_STAMP(0);

    // ---- A: projections.  Work item (t, sl): columns [64 t, +64) of [W_Q | W_KV], row slice sl.  A wavefront takes 64 rows:
    //      lane (g, rs = c / 8, piece c % 8) loads rows 32 rs + 8 g + 0..7 of its piece (whole 128-byte lines), transposed
    //      inside the lane.  The columns of an MFMA share their contraction rows, so each of the two row sets goes through
    //      the matrix unit with the other one's lanes zeroed.
    const int T = (CQ + 63) / 64, tA = w % T, slA = w / T;
    unsigned long long launches;
    Exchange x;
    {
        const int rs = c >> 3, piece = 8 * tA + (c & 7), qv = CQq / 8;
        const int r0 = slA * a.rows, rend = min(r0 + a.rows, a.D);
        const int row = r0 + 64 * wv + 32 * rs + 8 * g;                // (rows, D: multiples of eight)
        const bool live = slA < a.ksa && piece < CQ / 8 && row < rend;
        const bool isq = piece < qv;
        const size_t ld = isq ? qv : LR / 8;                           // row stride in pieces
        const h8 *wp = reinterpret_cast<const h8 *>(isq ? a.wq : a.wkv) + (live ? (size_t)row * ld + (isq ? piece : piece - qv) : 0);
        h8 wr[8], xa[2], f8[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) wr[u] = wp[live ? u * ld : 0];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int xr = r0 + 64 * wv + 32 * h + 8 * g;
            const bool on = c < B && xr < rend;
            const h8 xv = *reinterpret_cast<const h8 *>(a.x + (on ? (size_t)c * a.D + xr : 0));
            xa[h] = on ? xv : zero8;
        }
        asm volatile("s_load_dwordx2 %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)"
                     : "=s"(launches)
                     : "s"(a.counters + (size_t)w * kCounterStride)
                     : "memory");
        if (tid < R / 2) {
            const double inv_freq = exp2(-2.0 * (double)tid / (double)R * a.log2_base);
            cf::rope_cos_sin(a.pos, inv_freq, s_rope[tid], s_rope[R / 2 + tid]);
        }
        const unsigned long long cnt = launches + 1ull;
        x = Exchange{a.slots, 0, (uint32_t)(cnt + (cnt >> 32)), a.err, a.spin_ticks};
        transpose8(wr, f8);
        f32x4 acc[8];                                                  // [jj][rr]: batch row 4 g + rr, column 8 (c % 8) + jj
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) {
            acc[jj] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int h = 0; h < 2; ++h) acc[jj] = mfma16(xa[h], live && rs == h ? f8[jj] : zero8, acc[jj]);
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) acc[jj][rr] = ror8_add(acc[jj][rr]);
        }
        if (c < 8)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                float *dst = smem + (wv * 16 + 4 * g + rr) * 64 + 8 * c;
                *reinterpret_cast<f32x4 *>(dst) = f32x4{acc[0][rr], acc[1][rr], acc[2][rr], acc[3][rr]};
                *reinterpret_cast<f32x4 *>(dst + 4) = f32x4{acc[4][rr], acc[5][rr], acc[6][rr], acc[7][rr]};
            }
        lds_sync();
    }
    const Data X(a.data);
    const __amdgpu_buffer_rsrc_t r = cf::team::slots_rsrc(x);
    if (slA < a.ksa) {                                                 // (uniform)
        for (int i = tid; i < B * 64; i += NT) {
            const int b = i / 64, col = 64 * tA + i % 64;
            float sum = 0.f;
#pragma unroll
            for (int w8 = 0; w8 < NW; ++w8) sum += smem[w8 * 16 * 64 + i];
            if (col < CQ) X.st1(a.x1 + ((size_t)slA * B + b) * CQ + col, sum);
        }
        post(fA + slA * T + tA, x.stamp);
    }
    MLA_STAMP(1);           // A done

    // ---- B: member j of head `head`: columns [LJ*j, +LJ) of the up-projection (wavefront 0..3: 32 of the nope dimensions
    //      each, four 16-byte pieces of the rows), RoPE pairs 2j, 2j + 1 of the head's rotary query (wavefront 4).  Every
    //      wavefront waits for its sources itself and adds the row slices as it fetches them.
    {
        h8 wup[8];
        const int row = 32 * (wv & 3) + 8 * g;                         // (n: a multiple of eight)
        const bool mine = wv < 4 && row < a.n;
#pragma unroll
        for (int u = 0; u < 8; ++u)
            wup[u] = mine && c < 4 ? *reinterpret_cast<const h8 *>(a.wup + ((size_t)head * a.n + row + u) * L + LJ * j + c * 8) : zero8;
        const int ta = head * nr / 64, nt = (head * nr + nr - 1) / 64 - ta + 1;      // tiles of the head's columns: at most 4
        if (wv < 5) wait_flag(x, fA + min(lane / max(nt, 1), a.ksa - 1) * T + ta + lane % max(nt, 1), lane < nt * a.ksa);
        if (wv < 4) {
            float q8[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            const size_t src = a.x1 + (size_t)min(c, B - 1) * CQ + head * nr + (mine ? row : 0);
            f32x4 p[kMaxSlices][2];
#pragma unroll
            for (int k = 0; k < kMaxSlices; ++k)
#pragma unroll
                for (int h = 0; h < 2; ++h) p[k][h] = X.ld4(src + (size_t)min(k, a.ksa - 1) * B * CQ + 4 * h);
#pragma unroll
            for (int k = 0; k < kMaxSlices; ++k)
#pragma unroll
                for (int e = 0; e < 8; ++e) q8[e] += mine && k < a.ksa ? p[k][e >> 2][e & 3] : 0.f;
            h8 f8[8];
            const float m = row_max(max_abs(q8, 0.f));
            const int e = scale_exp(m);
            const Split<3> q = split_scaled<3>(q8, e, m);
            if (lane < 16) s_f[lane * NW + wv] = __builtin_amdgcn_ldexpf(1.f, -e);
            transpose8(wup, f8);
            f32x4 acc[8];
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) {
                acc[jj] = mfma16(q.part[0], f8[jj], f32x4{0.f, 0.f, 0.f, 0.f});
                acc[jj] = mfma16(q.part[1], f8[jj], acc[jj]);
                acc[jj] = mfma16(q.part[2], f8[jj], acc[jj]);
            }
            if (c < 4)
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) {
                    float *dst = smem + NW * 16 * 64 + (wv * 16 + 4 * g + rr) * LJ + 8 * c;      // (behind the sums of A)
                    *reinterpret_cast<f32x4 *>(dst) = f32x4{acc[0][rr], acc[1][rr], acc[2][rr], acc[3][rr]};
                    *reinterpret_cast<f32x4 *>(dst + 4) = f32x4{acc[4][rr], acc[5][rr], acc[6][rr], acc[7][rr]};
                }
        } else if (wv == 4) {
            // lane (batch row, k): k = 0, 1: the pairs' first elements, k = 2, 3: their partners
            const int b = lane >> 2, k = lane & 3, pr = 2 * j + (k & 1);
            float s = 0.f, p[kMaxSlices];
#pragma unroll
            for (int q = 0; q < kMaxSlices; ++q)
                p[q] = X.ld1(a.x1 + ((size_t)min(q, a.ksa - 1) * B + min(b, B - 1)) * CQ + head * nr + a.n + pr + (k >> 1) * (R / 2));
#pragma unroll
            for (int q = 0; q < kMaxSlices; ++q) s += q < a.ksa ? p[q] : 0.f;
            const float o = __shfl_xor(s, 2), cs = s_rope[pr], sn = s_rope[R / 2 + pr];
            const float v = k < 2 ? s * cs - o * sn : s * cs + o * sn;
            if (b < B) X.st1(a.xq + ((size_t)b * a.nh + head) * LR + L + pr + (k >> 1) * (R / 2), v);
        }
        lds_sync();
        MLA_STAMP(2);       // up-projection done
        {
            const int b = tid / LJ, cc = tid % LJ;
            const float *src = smem + NW * 16 * 64 + tid;
            const f32x4 f = *reinterpret_cast<const f32x4 *>(s_f + b * NW);
            const float sum = (src[0] * f[0] + src[16 * LJ] * f[1]) + (src[2 * 16 * LJ] * f[2] + src[3 * 16 * LJ] * f[3]);
            if (b < B) X.st1(a.xq + ((size_t)b * a.nh + head) * LR + LJ * j + cc, sum);
        }
        post(fB + head * TS + j, x.stamp);
    }
    MLA_STAMP(3);           // B done

    // ---- C: attention.  Work item (b, s, hg): cached rows [t0, t1) of batch row b against the queries of the heads
    //      [h0, h1).  A tile is 64 rows, read from memory once and kept in LDS for both products.  Scores: wavefront (dh, tq)
    //      takes 16 rows and 288 of the 576 dimensions, S^T = K Q^T as a 16 x 16 tile (rows = tokens, columns = heads),
    //      the query as a pair of fp16 operands (22 bits).  Online softmax per
    //      head over the 32 rows of one half of the tile, each half for itself (its four wavefronts hold the same state, so
    //      nothing but the scores goes through LDS).  Weighted sum: wavefront (th, kq) takes the latent dimensions
    //      [128 kq, +128) of the half th: A = probabilities (fp16), B = the rows, eight at a time transposed in the lane.
    const int ngroups = (a.nh + a.HG - 1) / a.HG;
    if (w < B * a.NS * ngroups) {                                      // one item per workgroup at most (the plan sees to it)
        const int hg = w % ngroups, b = w / ngroups / a.NS, s = w / ngroups % a.NS;
        const int h0 = hg * a.HG, h1 = min(h0 + a.HG, a.nh);           // the heads of this item
        const int t0 = min(s * a.tps, a.pos), t1 = min(t0 + a.tps, a.pos);
        h8 *qop_hi = reinterpret_cast<h8 *>(smem);                      // [kSteps][64]
        h8 *qop_lo = qop_hi + kQops;
        float *s_kn = smem + 2 * kQops * 4;                             // [LR] the new row
        float *s_sn = s_kn + LR;                                        // [NW][HT] its scores, a wavefront's steps each
        float *s_S = s_sn + NW * HT;                                         // [2][HT][SSTR] scores, per half of the dimensions
        float *s_ml = s_S + 2 * HT * SSTR;                              // [2][2][HT] maxima and sums of the two halves of the rows
        float *sO = s_ml + 4 * HT;                                      // [HT][L], at the end
        _Float16 *sK = reinterpret_cast<_Float16 *>(sO);                // [kTile][KSTR] cached rows
        // A thread carries nine 16-byte pieces of the tile, requested a tile ahead.  Rows past the range are read from its
        // last row (finite data) and get probability 0.
        constexpr int kPieces = kTile * (LR / 8) / NT;                  // 9
        const uint16_t *rows = a.cache + (size_t)b * a.max_seq * LR;
        h8 kr[kPieces];
        auto request = [&](int T0) {
#pragma unroll
            for (int k = 0; k < kPieces; ++k) {
                const int pc = tid + NT * k, row = pc / (LR / 8), col = pc % (LR / 8);
                kr[k] = *reinterpret_cast<const h8 *>(rows + (size_t)min(T0 + row, t1 - 1) * LR + 8 * col);
            }
        };
        if (t1 > t0) request(t0);                                       // (uniform) the rows do not wait for the query
        {
            const int nq = (h1 - h0) * TS;                              // at most 256
            wait_flag(x, fB + h0 * TS + min(tid, nq - 1), tid < nq);
            if (s == 0) {                                               // the new row's tiles: at most 10 x 4
                const int ta = CQq / 64, nt = (CQ - 1) / 64 - ta + 1, i = tid - 256;
                wait_flag(x, fA + (i >= 0 ? min(i / nt, a.ksa - 1) * T + ta + i % nt : 0), i >= 0 && i < nt * a.ksa);
            }
        }
        lds_sync();                                                     // (also: the sums of A and B have been read)
        asm volatile("" ::: "memory");
        MLA_STAMP(13);      // sources ready
        // query operands: entry e = (step m, lane (g2, head c2)) holds the eight dimensions score_dim(m, g2) + 0..7 of head c2,
        // scaled by log2(e) / sqrt(d_k), as fp16 pairs; heads outside the item's group are zero
        constexpr int NE = (kQops + NT - 1) / NT;
        f32x4 qv[NE][2];
#pragma unroll
        for (int k = 0; k < NE; ++k) {
            const int e = min(tid + NT * k, kQops - 1), m = e >> 6, g2 = (e >> 4) & 3, c2 = min(max(e & 15, h0), h1 - 1);
            const size_t src = a.xq + ((size_t)b * a.nh + c2) * LR + score_dim(m, g2);
            qv[k][0] = X.ld4(src);
            qv[k][1] = X.ld4(src + 4);
        }
        float qf[NE][8];                                                // this thread's entries in fp32, for the new token's score
        float kn[2] = {0.f, 0.f};
        if (s == 0)                                                     // (uniform)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int d = min(tid + NT * k, LR - 1);
                float p[kMaxSlices];
#pragma unroll
                for (int q = 0; q < kMaxSlices; ++q) p[q] = X.ld1(a.x1 + ((size_t)min(q, a.ksa - 1) * B + b) * CQ + CQq + d);
#pragma unroll
                for (int q = 0; q < kMaxSlices; ++q) kn[k] += q < a.ksa ? p[q] : 0.f;
            }
#pragma unroll
        for (int k = 0; k < NE; ++k) {
            const int e = tid + NT * k, c2 = e & 15;
#pragma unroll
            for (int i = 0; i < 8; ++i) qf[k][i] = c2 >= h0 && c2 < h1 ? qv[k][i >> 2][i & 3] * a.scale_log2e : 0.f;
            h8 hi, lo;
            split_hi_lo(qf[k], hi, lo);
            if (e < kQops) {
                qop_hi[e] = hi;
                qop_lo[e] = lo;
            }
        }
        if (s == 0) {
            // the new row: RoPE on the rotary part (dimension 512 + lane of wavefront 0), append (Sec. 2.1).  Its scores are
            // taken behind the tiles (in front of them these items were 3 us behind the others).
            const float o = __shfl_xor(kn[1], 32), cs = s_rope[lane & 31], sn = s_rope[R / 2 + (lane & 31)];
            kn[1] = lane < 32 ? kn[1] * cs - o * sn : kn[1] * cs + o * sn;
#pragma unroll
            for (int k = 0; k < 2; ++k)
                if (tid + NT * k < LR) {
                    s_kn[tid + NT * k] = kn[k];
                    if (hg == 0) a.cache[((size_t)b * a.max_seq + a.pos) * LR + tid + NT * k] = f2h(kn[k]);
                }
            if (t1 <= t0) lds_sync();                                   // (uniform; otherwise the tiles' barriers follow)
        }
        MLA_STAMP(4);           // query operands built
        const int th = wv >> 2, kq = wv & 3;                            // half of the tile rows, quarter of the latent dimensions
        float M = kNegBig, lw = 0.f;                                    // of head c: running maximum; sum over this lane's rows
        f32x4 O[8];                                                     // [jj][rr]: head 4 g + rr, dimension 128 kq + 8 c + jj
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) O[jj] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int T0 = t0; T0 < t1; T0 += kTile) {                       // uniform over the workgroup
#pragma unroll
            for (int k = 0; k < kPieces; ++k) {
                const int pc = tid + NT * k, row = pc / (LR / 8), col = pc % (LR / 8);
                *reinterpret_cast<h8 *>(sK + row * KSTR + 8 * col) = kr[k];
            }
            if (T0 + kTile < t1) request(T0 + kTile);
            lds_sync();
            {
                const int tq = wv & 3, dh = wv >> 2;
                const _Float16 *krow = sK + (16 * tq + c) * KSTR;
                f32x4 S0 = {0.f, 0.f, 0.f, 0.f}, S1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < kSteps / 2; ++i) {
                    const int m = dh * (kSteps / 2) + i;
                    const h8 ka = *reinterpret_cast<const h8 *>(krow + score_dim(m, g));
                    S0 = mfma16(ka, qop_hi[m * 64 + lane], S0);
                    S1 = mfma16(ka, qop_lo[m * 64 + lane], S1);
                }
                *reinterpret_cast<f32x4 *>(s_S + (dh * HT + c) * SSTR + 16 * tq + 4 * g) = S0 + S1;     // head c, tokens 16 tq + 4 g + 0..3
            }
            lds_sync();
            float sc[8], mx = kNegBig;                                  // head c, tokens 32 th + 8 g + 0..7 of the tile
            bool ok[8];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const float *src = s_S + c * SSTR + 32 * th + 8 * g + 4 * e;
                const f32x4 p = *reinterpret_cast<const f32x4 *>(src) + *reinterpret_cast<const f32x4 *>(src + HT * SSTR);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    ok[4 * e + i] = T0 + 32 * th + 8 * g + 4 * e + i < t1;
                    sc[4 * e + i] = ok[4 * e + i] ? p[i] : kNegBig;
                    mx = fmaxf(mx, sc[4 * e + i]);
                }
            }
            mx = cf::lanes::max_groups<16>(mx);
            const float Mn = fmaxf(M, mx);
            if (__any(Mn > M)) {                                        // a maximum has grown: rescale
                const float f = __builtin_amdgcn_exp2f(M - Mn);
                lw *= f;
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) {
                    const float fr = __shfl(f, 4 * g + rr);             // factor of the heads this lane accumulates
#pragma unroll
                    for (int jj = 0; jj < 8; ++jj) O[jj][rr] *= fr;
                }
                M = Mn;
            }
            h8 pa;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float pw = ok[i] ? __builtin_amdgcn_exp2f(sc[i] - Mn) : 0.f;
                pa[i] = (_Float16)pw;
                lw += pw;
            }
            {
                h8 vr[8], f8[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) vr[u] = *reinterpret_cast<const h8 *>(sK + (32 * th + 8 * g + u) * KSTR + 128 * kq + 8 * c);
                transpose8(vr, f8);
#pragma unroll
                for (int jj = 0; jj < 8; ++jj) O[jj] = mfma16(pa, f8[jj], O[jj]);
            }
            lds_sync();                                                 // the tile is consumed: the next one may land
        }
        MLA_STAMP(11);          // rows consumed
        if (s == 0) {
            // score of the new token (neither its row nor the query is rounded): wavefront wv takes the operand steps wv,
            // wv + 8, ..., whose entries its lanes have built
            float d = 0.f;
#pragma unroll
            for (int k = 0; k < NE; ++k)
                if (wv + NW * k < kSteps) {                             // (uniform)
                    const f32x4 *kd = reinterpret_cast<const f32x4 *>(s_kn + score_dim(wv + NW * k, g));
#pragma unroll
                    for (int i = 0; i < 8; ++i) d = fmaf(qf[k][i], kd[i >> 2][i & 3], d);
                }
            d = cf::lanes::sum_groups<16>(d);
            if (lane < HT) s_sn[wv * HT + c] = d;
        }
        // the two halves (and the new token) -> one partial (m, l, acc) per head
        lw = cf::lanes::sum_groups<16>(lw);
        if (kq == 0 && lane < HT) {
            s_ml[th * 2 * HT + c] = M;
            s_ml[th * 2 * HT + HT + c] = lw;
        }
        if (th == 1) {
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                float *dst = sO + (4 * g + rr) * L + 128 * kq + 8 * c;
                *reinterpret_cast<f32x4 *>(dst) = f32x4{O[0][rr], O[1][rr], O[2][rr], O[3][rr]};
                *reinterpret_cast<f32x4 *>(dst + 4) = f32x4{O[4][rr], O[5][rr], O[6][rr], O[7][rr]};
            }
        }
        lds_sync();
        if (th == 0) {
            const size_t dst = a.x3 + (size_t)w * HT * L;
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const int h = 4 * g + rr;
                if (h >= h0 && h < h1) {
                    float sn = kNegBig;
                    if (s == 0) {
                        sn = s_sn[h];
#pragma unroll
                        for (int w8 = 1; w8 < NW; ++w8) sn += s_sn[w8 * HT + h];
                    }
                    const float M0 = s_ml[h], M1 = s_ml[2 * HT + h], Mx = fmaxf(fmaxf(M0, M1), sn);
                    const float f0 = __builtin_amdgcn_exp2f(M0 - Mx), f1 = __builtin_amdgcn_exp2f(M1 - Mx);
                    const float fn = s == 0 ? __builtin_amdgcn_exp2f(sn - Mx) : 0.f;
                    const float *src = sO + h * L + 128 * kq + 8 * c;
                    f32x4 o[2];
#pragma unroll
                    for (int jj = 0; jj < 8; ++jj) o[jj >> 2][jj & 3] = O[jj][rr] * f0 + src[jj] * f1;
                    if (s == 0)
#pragma unroll
                        for (int jj = 0; jj < 8; ++jj) o[jj >> 2][jj & 3] = fmaf(s_kn[128 * kq + 8 * c + jj], fn, o[jj >> 2][jj & 3]);
                    X.st4(dst + (size_t)h * L + 128 * kq + 8 * c, o[0]);
                    X.st4(dst + (size_t)h * L + 128 * kq + 8 * c + 4, o[1]);
                    if (kq == 0 && c == 0) {
                        X.st1(a.xml + ((size_t)w * HT + h) * 2, Mx);
                        X.st1(a.xml + ((size_t)w * HT + h) * 2 + 1, s_ml[HT + h] * f0 + s_ml[3 * HT + h] * f1 + fn);
                    }
                }
            }
        }
        post(fC + w, x.stamp);
    }
    MLA_STAMP(5);           // C done

    // ---- D: merge latent dimensions [LJ*j, +LJ) of head `head` over the token ranges (online softmax, Alg. 4 steps 8-10).
    //      The weights of E1 are requested first: W_Down[head], wavefront wv: rows [64 wv, +64); W_O, rows of the head, column
    //      block j, wavefront wv: rows [32 (wv % 4), +32).
    const int dpE = a.D / 8, pcsE = (dpE + TS - 1) / TS;                // 16-byte pieces of an output row; per member (<= 16)
    h8 wdn[16], wor[8];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int row = 64 * wv + 32 * (u >> 3) + 8 * g + (u & 7);
        wdn[u] = c < a.v / 8 ? *reinterpret_cast<const h8 *>(a.wdown + ((size_t)head * L + row) * a.v + c * 8) : zero8;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const int row = 32 * (wv & 3) + 8 * g + u, piece = j * pcsE + c;
        wor[u] = c < pcsE && piece < dpE && row < a.v
                     ? *reinterpret_cast<const h8 *>(a.wo + ((size_t)head * a.v + row) * a.D + piece * 8)
                     : zero8;
    }
    {
        const int hgr = head / a.HG, ni = B * a.NS;                     // ni <= 256 sources
        wait_flag(x, fC + min(tid, ni - 1) * ngroups + hgr, tid < ni);
        lds_sync();
        asm volatile("" ::: "memory");
        MLA_STAMP(12);      // sources ready
        // half-wavefront = batch row; lane s of it: maximum and sum of range s; and (sq, d4): four dimensions of every
        // fourth range
        const int b = tid >> 5, l5 = tid & 31, sq = l5 >> 3, d4 = l5 & 7, bb = min(b, B - 1);
        const size_t it0 = (size_t)bb * a.NS * ngroups + hgr;           // item of range 0; ngroups further per range
        const size_t ml = a.xml + ((it0 + (size_t)min(l5, a.NS - 1) * ngroups) * HT + head) * 2;
        float m = X.ld1(ml), l = X.ld1(ml + 1);
        f32x4 p[kMaxSplits / 4];
#pragma unroll
        for (int k = 0; k < kMaxSplits / 4; ++k) {
            p[k] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (4 * k < a.NS)                                           // (uniform)
                p[k] = X.ld4(a.x3 + ((it0 + (size_t)min(sq + 4 * k, a.NS - 1) * ngroups) * HT + head) * L + LJ * j + 4 * d4);
        }
        if (l5 >= a.NS) m = kNegBig, l = 0.f;
        const float M = cf::lanes::max_half(m);
        const float f = l5 < a.NS ? __builtin_amdgcn_exp2f(m - M) : 0.f, Ls = cf::lanes::sum_half(l * f);
        f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < kMaxSplits / 4; ++k) {
            const float fk = __shfl(f, (lane & 32) + sq + 4 * k);       // 0 past the ranges
#pragma unroll
            for (int i = 0; i < 4; ++i) z[i] = fmaf(p[k][i], fk, z[i]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            z[i] = cf::lanes::add16(z[i] + cf::lanes::xor8(z[i])) / Ls;
        }
        if (sq == 0 && b < B) X.st4(a.xz + ((size_t)b * a.nh + head) * L + LJ * j + 4 * d4, z);
        post(fD + head * TS + j, x.stamp);
    }
    MLA_STAMP(6);           // z posted

    // ---- E1: a_head = z W_Down[head] (contraction over 512: 64 rows per wavefront, added through LDS), then the rows of
    //      W_O that belong to this head (contraction over v <= 128: wavefront (part, st) 32 rows, part: first and third, or
    //      second, of the fp16 parts of a), column block j of the output
    {
        float *s_a = smem, *s_red = smem + 16 * AS;                     // [16][AS], [NW][16][128]
        wait_flag(x, fD + head * TS + min(lane, TS - 1), lane < TS);
        f32x4 zv[2][2];
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
            for (int h = 0; h < 2; ++h) zv[st][h] = X.ld4(a.xz + ((size_t)min(c, B - 1) * a.nh + head) * L + 64 * wv + 32 * st + 8 * g + 4 * h);
        f32x4 acc[8];
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) acc[jj] = f32x4{0.f, 0.f, 0.f, 0.f};
        float v[2][8], vmax = 0.f;
#pragma unroll
        for (int st = 0; st < 2; ++st) {
#pragma unroll
            for (int i = 0; i < 8; ++i) v[st][i] = zv[st][i >> 2][i & 3];
            vmax = max_abs(v[st], vmax);
        }
        vmax = row_max(vmax);
        const int ez = scale_exp(vmax);
#pragma unroll
        for (int st = 0; st < 2; ++st) {
            h8 f8[8];
            const Split<3> z = split_scaled<3>(v[st], ez, vmax);
            transpose8(wdn + 8 * st, f8);
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) {
                acc[jj] = mfma16(z.part[0], f8[jj], acc[jj]);
                acc[jj] = mfma16(z.part[1], f8[jj], acc[jj]);
                acc[jj] = mfma16(z.part[2], f8[jj], acc[jj]);
            }
        }
        // the wavefronts' partial products with the inverse of their rows' scales, and their sum
        auto spill = [&](int e) {
            if (lane < 16) s_f[lane * NW + wv] = __builtin_amdgcn_ldexpf(1.f, -e);
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                float *dst = s_red + (wv * 16 + 4 * g + rr) * 128 + 8 * c;
                *reinterpret_cast<f32x4 *>(dst) = f32x4{acc[0][rr], acc[1][rr], acc[2][rr], acc[3][rr]};
                *reinterpret_cast<f32x4 *>(dst + 4) = f32x4{acc[4][rr], acc[5][rr], acc[6][rr], acc[7][rr]};
            }
        };
        auto total = [&](int i) {
            const f32x4 f[2] = {*reinterpret_cast<const f32x4 *>(s_f + i / 128 * NW), *reinterpret_cast<const f32x4 *>(s_f + i / 128 * NW + 4)};
            float sum = 0.f;
#pragma unroll
            for (int w8 = 0; w8 < NW; ++w8) sum = fmaf(s_red[w8 * 16 * 128 + i], f[w8 >> 2][w8 & 3], sum);
            return sum;
        };
        spill(ez);
        lds_sync();
        for (int i = tid; i < 16 * 128; i += NT) s_a[i / 128 * AS + i % 128] = total(i);
        lds_sync();
        MLA_STAMP(8);           // a_head ready
        {
            const int st = wv & 3;
            float v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = s_a[c * AS + 32 * st + 8 * g + i];
            h8 f8[8];
            const float m = row_max(max_abs(v, 0.f));
            const int e = scale_exp(m);
            const Split<3> q = split_scaled<3>(v, e, m);
            transpose8(wor, f8);
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) acc[jj] = mfma16(wv < 4 ? q.part[0] : q.part[1], f8[jj], f32x4{0.f, 0.f, 0.f, 0.f});
            if (wv < 4)
#pragma unroll
                for (int jj = 0; jj < 8; ++jj) acc[jj] = mfma16(q.part[2], f8[jj], acc[jj]);
            spill(e);
        }
        lds_sync();
        for (int i = tid; i < B * 128; i += NT) {
            const int b = i / 128, cc = i % 128, col = j * pcsE * 8 + cc;
            if (cc < 8 * pcsE && col < a.D) cf::team::put(r, ((size_t)head * B + b) * a.D + col, total(i), x.stamp);
        }
    }
    MLA_STAMP(10);          // E1 done

    // ---- E2: sum over the heads (what the paper does with atomicAdd), columns [CW*w, +CW) of the output: thread (quarter,
    //      value): the value's partials of four heads
    {
        const int CW = (a.D + a.W - 1) / a.W, nv = B * CW;             // CW <= 8, nv <= 128
        float *s_o = smem;                                              // [4][128] (a_head has been read)
        const int qtr = tid >> 7, v = tid & 127, b = v / CW, col = CW * w + v % CW;
        const bool on = v < nv && col < a.D;
        pair_t q[4];
        long long tw = 0;
        for (;;) {
#pragma unroll
            for (int k = 0; k < 4; ++k) q[k] = cf::team::peek(r, on ? ((size_t)min(4 * qtr + k, a.nh - 1) * B + b) * a.D + col : 0);
            __builtin_amdgcn_sched_barrier(0);
            bool ok = true;
#pragma unroll
            for (int k = 0; k < 4; ++k) ok &= q[k].y == x.stamp;
            if (!on || ok || cf::team::gave_up(x, tw)) break;
        }
        float sum = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) sum += 4 * qtr + k < a.nh ? __builtin_bit_cast(float, q[k].x) : 0.f;
        s_o[tid] = sum;
        lds_sync();
        if (qtr == 0 && on) a.out[(size_t)b * a.D + col] = f2h((s_o[v] + s_o[128 + v]) + (s_o[256 + v] + s_o[384 + v]));
    }
    if (tid == 0) a.counters[(size_t)w * kCounterStride] = launches + 1ull;
    MLA_STAMP(9);
#if CF_STAMPS
    lds_sync();
    if (tid < kMlaStamps && w < 256) g_mla_ts[w * kMlaStamps + tid] = s_ts[tid];
#endif
}

}  // namespace

struct cf_mla_s {
    cf_mla_config cfg;
    int W = 0;
    char *ws = nullptr;
    size_t ws_bytes = 0, clear_bytes = 0;            // clear_bytes: counters, flags and stamped slots, at the front
    uint64_t *slots = nullptr, *hslots = nullptr;    // stamped slots of the token-range kernel, of the head-team kernel
    float *data = nullptr;          // values of the token-range kernel's other hand-overs
    uint32_t *flags = nullptr;      // their flags
    float *qdbg = nullptr, *zpart = nullptr;
    unsigned long long *counters = nullptr;
    uint32_t *err = nullptr;
    size_t x1 = 0, xq = 0, x3 = 0, xml = 0, xz = 0;
    long long spin_ticks = 200000000LL;
    int max_splits = 0;             // 0: chosen by the library
    int last_batch = 0;
    bool last_heads = false;        // the last call ran the head-team kernel
    int last_hip = 0;
};

namespace {

// 64-column tiles of [W_Q | W_KV] (those of W_Q are rounded up: W_KV fills nine)
int tiles_of(const cf_mla_config &c) { return (c.n_heads * (c.nope_dim + R) + 63) / 64 + LR / 64; }

// token ranges of a call: NS ranges of tps cached rows per batch row; and the heads per attention item: as few as
// the number of workgroups allows (an item fetches the queries and publishes the partial results of its heads only:
// per workgroup that traffic, not the arithmetic, is what takes time)
void plan_splits(const cf_mla_s *t, int batch, int pos, int *ns, int *tps, int *hg)
{
    int cap = t->W / batch;
    cap = cap < 1 ? 1 : cap > kMaxSplits ? kMaxSplits : cap;
    if (t->max_splits > 0 && t->max_splits < cap) cap = t->max_splits;
    int per = (pos + cap - 1) / cap;
    per = (per + 15) / 16 * 16;
    if (per < 64 && t->max_splits == 0) per = 64;     // below a tile more ranges only add partials
    if (per < 16) per = 16;
    *tps = per;
    const int n = (pos + per - 1) / per;
    *ns = n < 1 ? 1 : n;                              // range 0 always exists: it scores the new token
    int groups = 1;
    while (2 * groups <= t->cfg.n_heads && batch * *ns * 2 * groups <= t->W) groups *= 2;
    *hg = (t->cfg.n_heads + groups - 1) / groups;
}

}  // namespace

extern "C" {

int cf_mla_create(const cf_mla_config *cfg, cf_mla *out)
{
    if (!cfg || !out) return CF_EINVAL;
    *out = nullptr;
    const cf_mla_config &c = *cfg;
    if (c.d_model < 16 || c.n_heads < 1 || c.nope_dim < 1 || c.v_head_dim < 1 || c.max_batch < 1 || c.max_seq < 1 ||
        !(c.rope_base > 1.f))
        return CF_EINVAL;
    // what the kernel is written for
    const int W = c.n_heads * TS;
    const int CQq = c.n_heads * (c.nope_dim + R);
    if (c.kv_lora_rank != L || c.rope_dim != R || c.max_batch > MAXBATCH || c.n_heads > HT || c.d_model % 32 ||
        c.d_model > 16 * NT || c.v_head_dim % 8 || c.v_head_dim > 128 || c.nope_dim % 8 || c.nope_dim > 128 || c.d_model > 8 * W)
        return CF_EUNSUPPORTED;
    int ksa = 0, rows = 0;
    if (!cf::mla::slices(c, &ksa, &rows)) return CF_EUNSUPPORTED;
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return CF_EHIP;
    if (W > prop.multiProcessorCount) return CF_EUNSUPPORTED;        // all workgroups resident, one per compute unit
    const size_t lds = kLdsFloats * sizeof(float);
    int per_cu = 0;
    const void *fn = reinterpret_cast<const void *>(fused_mla_decode);
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, NT, lds) != hipSuccess || per_cu < 1)
        return CF_EUNSUPPORTED;
    if (!cf::mla::heads_prepare()) return CF_EUNSUPPORTED;
    cf_mla t = new (std::nothrow) cf_mla_s();
    if (!t) return CF_ENOMEM;
    t->cfg = c;
    t->W = W;
    const size_t B = c.max_batch, CQ = (size_t)CQq + LR, nh = c.n_heads;
    t->x1 = 0;
    t->xq = t->x1 + (size_t)kMaxSlices * B * CQ;
    t->x3 = t->xq + B * nh * LR;                                  // (an item per workgroup at most)
    t->xml = t->x3 + (size_t)W * HT * L;
    t->xz = t->xml + (size_t)W * HT * 2;
    const size_t ndata = t->xz + B * nh * L;
    size_t hfirst[3];
    // every kind of hand-over has memory of its own: a flag or a stamp never lies where other data has been
    const size_t nslots = B * nh * c.d_model, nhslots = cf::mla::heads_layout(c, hfirst);
    auto up = [](size_t v) { return (v + 255) / 256 * 256; };
    const size_t head_b = up(256 + (size_t)W * kCounterStride * sizeof(unsigned long long)), flag_b = 4 * 256 * sizeof(uint32_t);
    const size_t slot_b = up(nslots * 8), hslot_b = up(nhslots * 8), data_b = up(ndata * 4), q_b = up(nh * LR * 4);
    t->clear_bytes = head_b + flag_b + slot_b + hslot_b;
    t->ws_bytes = t->clear_bytes + data_b + q_b + nh * TS * (2 + L) * sizeof(float);
    if (slot_b > 0xfffffff0ull || data_b > 0xfffffff0ull) {
        delete t;
        return CF_EUNSUPPORTED;
    }
    hipError_t e = hipMalloc(reinterpret_cast<void **>(&t->ws), t->ws_bytes);
    if (e == hipSuccess) e = hipMemset(t->ws, 0, t->clear_bytes);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) {
        if (t->ws) (void)hipFree(t->ws);
        delete t;
        return e == hipErrorOutOfMemory ? CF_ENOMEM : CF_EHIP;
    }
    t->err = reinterpret_cast<uint32_t *>(t->ws + 128);
    t->counters = reinterpret_cast<unsigned long long *>(t->ws + 256);
    char *cur = t->ws + head_b;
    t->flags = reinterpret_cast<uint32_t *>(cur);
    t->slots = reinterpret_cast<uint64_t *>(cur += flag_b);
    t->hslots = reinterpret_cast<uint64_t *>(cur += slot_b);
    t->data = reinterpret_cast<float *>(cur += hslot_b);
    t->qdbg = reinterpret_cast<float *>(cur += data_b);
    t->zpart = reinterpret_cast<float *>(cur += q_b);
    *out = t;
    return CF_OK;
}

int cf_mla_destroy(cf_mla t)
{
    if (!t) return CF_EINVAL;
    hipError_t e = hipFree(t->ws);
    delete t;
    return e == hipSuccess ? CF_OK : CF_EHIP;
}

int cf_mla_decode(cf_mla t, int32_t batch, const void *x, const void *W_q, const void *W_kv, const void *W_up,
                  const void *W_down, const void *W_o, void *kv_cache, int32_t pos, void *out, void *stream)
{
    if (!t || !x || !W_q || !W_kv || !W_up || !W_down || !W_o || !kv_cache || !out) return CF_EINVAL;
    if (batch < 1 || batch > t->cfg.max_batch || pos < 0 || pos >= t->cfg.max_seq) return CF_EINVAL;
    const void *ptrs[] = {x, W_q, W_kv, W_up, W_down, W_o, kv_cache, out};
    for (const void *p : ptrs)
        if (reinterpret_cast<uintptr_t>(p) & 15u) return CF_EINVAL;
    const cf_mla_config &c = t->cfg;
    if (batch <= kHeadsBatch && t->max_splits == 0) {
        // the head-team kernel (every head scans the cached rows itself; see cf_mla_heads.hip)
        cf::mla::HeadsArgs h;
        std::memset(&h, 0, sizeof h);
        h.x = static_cast<const uint16_t *>(x);
        h.wq = static_cast<const uint16_t *>(W_q);
        h.wkv = static_cast<const uint16_t *>(W_kv);
        h.wup = static_cast<const uint16_t *>(W_up);
        h.wdown = static_cast<const uint16_t *>(W_down);
        h.wo = static_cast<const uint16_t *>(W_o);
        h.cache = static_cast<uint16_t *>(kv_cache);
        h.out = static_cast<uint16_t *>(out);
        h.qdbg = t->qdbg, h.zpart = t->zpart;
        h.slots = t->hslots, h.counters = t->counters, h.err = t->err;
        size_t first[3];
        (void)cf::mla::heads_layout(c, first);
        h.x1 = first[0], h.x3 = first[1], h.x6 = first[2];
        h.D = c.d_model, h.nh = c.n_heads, h.n = c.nope_dim, h.v = c.v_head_dim, h.pos = pos, h.W = t->W;
        (void)cf::mla::slices(c, &h.ksa, &h.rows);
        h.tiles = tiles_of(c), h.CW = (c.d_model + t->W - 1) / t->W;
        h.div_t = cf::divisor(h.tiles), h.div_cw = cf::divisor(h.CW);
        h.scale_log2e = 1.4426950408889634f / std::sqrt((float)(c.nope_dim + R));
        h.log2_base = std::log2((double)c.rope_base);
        h.spin_ticks = t->spin_ticks;
        t->last_batch = batch, t->last_heads = true;
        const int e = cf::mla::heads_launch(h, stream);
        if (e != (int)hipSuccess) {
            t->last_hip = e;
            return CF_EHIP;
        }
        return CF_OK;
    }
    MlaArgs a;
    std::memset(&a, 0, sizeof a);
    a.x = static_cast<const uint16_t *>(x);
    a.wq = static_cast<const uint16_t *>(W_q);
    a.wkv = static_cast<const uint16_t *>(W_kv);
    a.wup = static_cast<const uint16_t *>(W_up);
    a.wdown = static_cast<const uint16_t *>(W_down);
    a.wo = static_cast<const uint16_t *>(W_o);
    a.cache = static_cast<uint16_t *>(kv_cache);
    a.out = static_cast<uint16_t *>(out);
    a.slots = t->slots, a.data = t->data, a.flags = t->flags;
    a.counters = t->counters;
    a.err = t->err;
    // the exchange areas are laid out for max_batch; a smaller batch uses the front of each
    a.x1 = t->x1, a.xq = t->xq, a.x3 = t->x3, a.xml = t->xml, a.xz = t->xz;
    a.D = c.d_model, a.nh = c.n_heads, a.n = c.nope_dim, a.v = c.v_head_dim, a.B = batch, a.pos = pos;
    a.max_seq = c.max_seq, a.W = t->W;
    plan_splits(t, batch, pos, &a.NS, &a.tps, &a.HG);
    (void)cf::mla::slices(c, &a.ksa, &a.rows);
    a.scale_log2e = 1.4426950408889634f / std::sqrt((float)(c.nope_dim + R));
    a.log2_base = std::log2((double)c.rope_base);
    a.spin_ticks = t->spin_ticks;
    t->last_batch = batch, t->last_heads = false;
    hipLaunchKernelGGL(fused_mla_decode, dim3(t->W), dim3(NT), kLdsFloats * sizeof(float), static_cast<hipStream_t>(stream), a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        t->last_hip = (int)e;
        return CF_EHIP;
    }
    return CF_OK;
}

int cf_mla_status(cf_mla t, void *stream)
{
    if (!t) return CF_EINVAL;
    hipError_t e = hipStreamSynchronize(static_cast<hipStream_t>(stream));
    uint32_t flag = 0;
    if (e == hipSuccess) e = hipMemcpy(&flag, t->err, sizeof flag, hipMemcpyDeviceToHost);
    if (e != hipSuccess) {
        t->last_hip = (int)e;
        return CF_EHIP;
    }
    if (flag) {
        e = hipMemset(t->ws, 0, t->clear_bytes);     // launch counters and all stamps start afresh
        if (e == hipSuccess) e = hipDeviceSynchronize();
        return e == hipSuccess ? CF_ETIMEOUT : CF_EHIP;
    }
    return CF_OK;
}

int cf_mla_set_splits(cf_mla t, int32_t max_splits)
{
    if (!t || max_splits < 0 || max_splits > kMaxSplits) return CF_EINVAL;
    t->max_splits = max_splits;
    return CF_OK;
}

int cf_mla_debug_export(cf_mla t, int32_t what, void *host_dst, size_t bytes, void *stream)
{
    if (!t || !host_dst || what < 0 || what > 2 || t->last_batch < 1) return CF_EINVAL;
    const size_t B = t->last_batch, nh = t->cfg.n_heads;
    const size_t per = what == 1 ? R : L;
    if (bytes != B * nh * per * sizeof(float)) return CF_EINVAL;
    hipError_t e = hipStreamSynchronize(static_cast<hipStream_t>(stream));
    float *dst = static_cast<float *>(host_dst);
    if (e == hipSuccess && what == 2 && t->last_heads) {
        // the head-team kernel merges behind W_Down: z is put together here from the members' partials, a head at a time (on
        // the stack: nothing in here may throw)
        float part[TS][2 + L];
        for (size_t h = 0; e == hipSuccess && h < nh; ++h) {
            e = hipMemcpy(part, t->zpart + h * TS * (2 + L), sizeof part, hipMemcpyDeviceToHost);
            float M = part[0][0];
            for (int s = 1; s < TS; ++s) M = std::fmax(M, part[s][0]);
            double f[TS], ls = 0.0;
            for (int s = 0; s < TS; ++s) {
                f[s] = std::exp2((double)part[s][0] - M);
                ls += f[s] * part[s][1];
            }
            for (int d = 0; d < L; ++d) {
                double z = 0.0;
                for (int s = 0; s < TS; ++s) z += f[s] * part[s][2 + d];
                dst[h * L + d] = (float)(z / ls);
            }
        }
    } else if (e == hipSuccess && what == 2) {
        // z of the last call still sits in its exchange area, [b][head][L]
        e = hipMemcpy(dst, t->data + t->xz, bytes, hipMemcpyDeviceToHost);
    } else if (e == hipSuccess) {
        // the query: [b][head][L + R], of the token-range kernel still in its exchange area
        const float *q = (t->last_heads ? t->qdbg : t->data + t->xq) + (what == 1 ? L : 0);
        e = hipMemcpy2D(dst, per * sizeof(float), q, LR * sizeof(float), per * sizeof(float), B * nh, hipMemcpyDeviceToHost);
    }
    if (e != hipSuccess) {
        t->last_hip = (int)e;
        return CF_EHIP;
    }
    return CF_OK;
}

#if CF_STAMPS
// profiling library only: the stage stamps of the last launch (host buffer of 256 * 16 64-bit words)
int cf_mla_trace_read(void *host_dst)
{
    hipError_t e = hipDeviceSynchronize();
    if (e == hipSuccess) e = hipMemcpyFromSymbol(host_dst, HIP_SYMBOL(g_mla_ts), sizeof(unsigned long long) * 256 * kMlaStamps);
    return e == hipSuccess ? CF_OK : CF_EHIP;
}
#endif

int cf_mla_set_spin_limit(cf_mla t, int32_t spin_limit_us)
{
    if (!t || spin_limit_us < 0) return CF_EINVAL;
    t->spin_ticks = (long long)spin_limit_us * 100;
    return CF_OK;
}

int64_t cf_mla_algorithmic_bytes(const cf_mla_config *c, int32_t batch, int32_t pos)
{
    if (!c) return 0;
    const int64_t nr = c->nope_dim + c->rope_dim, lr = c->kv_lora_rank + c->rope_dim, B = batch;
    const int64_t weights = (int64_t)c->d_model * (c->n_heads * nr + lr) + (int64_t)c->n_heads * c->nope_dim * c->kv_lora_rank +
                            (int64_t)c->n_heads * c->kv_lora_rank * c->v_head_dim + (int64_t)c->n_heads * c->v_head_dim * c->d_model;
    return 2 * (weights + B * (int64_t)pos * lr + B * lr + 2 * B * c->d_model);
}

}  // extern "C"
