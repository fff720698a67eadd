// Fused MLA decode step at batch 1 (paper Appendix B, Alg. 4) with the HEAD as the unit of work, the way Alg. 4 assigns
// a cluster to a head: 16 co-resident workgroups per head, every member scans 1/16 of the cached rows for its head with
// vector arithmetic.  Every head reads every cached row, which the last-level cache absorbs at one batch row; from
// batch 2 on the kernel of cf_mla.hip (token ranges as the unit of work, MFMA tiles over all heads) is the faster one,
// and cf_mla_decode picks between the two.
//
// The step is bound by its hand-overs through memory, not by its 32 MB, so the work is cut to need three of them where
// Alg. 4 has six collectives.  What a head's members would have to exchange in between they compute redundantly, each
// from the whole weight block of the head (2 x 131 KB, which the L2 of the head's die serves to its 16 members):
//
//   A   projections        [q | kv_new] = x [W_Q | W_KV]    64 columns x 1/4 of the rows per workgroup
//   -- hand-over: q_i to the members of head i, kv_new to the last member of every head
//   B   up-projection      q_lat_i = q_nope_i W_Up[i]       every member for itself, all of W_Up[i]
//   C   attention          partial softmax over 1/16 of the tokens: (m, l, acc[kv_lora_rank]) in LDS; the last member
//                          appends the new row and counts the new token
//   D   down-projection    (m, l, acc W_Down[i])            of the member's own partial, all of W_Down[i]: the merge of
//                          the partials is linear, so it can follow the product: v_head_dim values to hand over, not 512
//   -- hand-over: the 16 partials of head i to its members
//   E1  merge (Alg. 4 steps 8-10), rows of W_O of head i, 1/16 of the output columns per member: a partial of out per head
//   -- hand-over: the heads' partials
//   E2  sum over heads     every workgroup: 1/W of the output columns (the paper's atomicAdd)
//
// DeepSeek-V2-Lite shape, 4096 rows, weights and rows from memory: 21.1 us a step (21.9 with conditions around loads, which waited
// for the first load of a group before the next went out, and with both batches of rows requested in front of the product that
// needs W_Up: a wavefront stands still while its loads are accepted; 22.6 with shuffles between lanes instead
// of permlane swaps; 27.9 with five hand-overs: partial
// sums of the projections, latent query, partials, partial a_i, partial out); 100 rows 17.5 us (18.6), 16000 rows 35.4 (46.7).  Stages, us from kernel
// start, mean / latest workgroup, launches back to back: projections posted 3.0 / 4.1, q arrived 6.8 / 7.6, query ready 8.3 / 9.4, rows used
// 11.3 / 12.2, partial folded 13.8 / 14.7, D posted 14.7 / 15.5, a_i ready 17.5 / 18.3, partial out posted 17.9 / 18.7, end 19.4 / 19.9.  What
// bounds it is this chain: the three hand-overs take 5.4 us from the latest post to the mean arrival, waiting for the latest post 2.7, the
// stages 11.3, bound by what a compute unit loads (64 KB of A, 131 KB of W_Up, 295 KB of rows, 131 KB of W_Down): requesting W_Up or the
// rows in front of the first hand-over moves the wait, not the end (21.2 - 21.9 us).
// All waits are bounded (CF_ETIMEOUT), all workgroups have to be resident at once.
#include "cf_lanes_device.h"
#include "cf_mla_internal.h"
#include "cf_rope_device.h"
#include "cf_stream_device.h"
#include "cf_team_device.h"

namespace {

using cf::team::Exchange;
using cf::team::pair_t;
constexpr int NT = 512;             // threads per workgroup
constexpr int NW = NT / 64;
constexpr int TS = 16;              // workgroups per head (team)
constexpr int L = 512;              // kv_lora_rank the lane mapping is written for: 16 lanes x 32 values per cached row
constexpr int R = 64;               // rope_dim: 16 lanes x 4 values
constexpr int LR = L + R;
constexpr int kMaxSlices = 4;       // row slices of the projections at most
constexpr int VS = 130;             // slots of a member's partial: m, l, v_head_dim <= 128 values
constexpr int kCounterStride = 16;
constexpr int PSTR = L + 8;         // floats of a wavefront's attention partial in LDS: m, l, pad, acc[L]
constexpr size_t kDynLds = (size_t)NW * PSTR * sizeof(float);   // also [NW][L] sums of B, [NW][128] of D, 512 + [NW][128] of E1
constexpr float kNegBig = -1.0e30f;

using cf::h8;
using cf::kNoLoad;
using Weights = cf::Part<0>;
typedef _Float16 h4 __attribute__((ext_vector_type(4)));


__device__ __forceinline__ uint16_t f2h(float f) { return __builtin_bit_cast(uint16_t, (_Float16)f); }

namespace lanes = cf::lanes;

// Workgroup barrier that orders LDS accesses only (__syncthreads() would also wait until the write-through stores of
// the last hand-over have reached memory); nothing here passes data between the threads of a workgroup through
// global memory.
__device__ __forceinline__ void lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Stage time stamps of every workgroup, only in builds with -DCF_STAMPS=1 (the profiling library).
#ifndef CF_STAMPS
#define CF_STAMPS 0
#endif
#if CF_STAMPS
constexpr int kMlaStamps = 16;
__device__ unsigned long long g_heads_ts[256 * kMlaStamps];
#define MLA_STAMP(k) do { if (threadIdx.x == 0) s_ts[k] = wall_clock64(); } while (0)
#else
#define MLA_STAMP(k)
#endif

// The stamped value at idx (one poll per try).
__device__ __forceinline__ float take1(const Exchange &x, __amdgpu_buffer_rsrc_t r, size_t idx)
{
    long long t0 = 0;
    for (;;) {
        const pair_t q = cf::team::peek(r, idx);
        if (q.y == x.stamp) return __builtin_bit_cast(float, q.x);
        if (cf::team::gave_up(x, t0)) return 0.f;
    }
}

__global__ void __launch_bounds__(NT) fused_mla_heads(const cf::mla::HeadsArgs a)
{
    extern __shared__ __align__(16) float s_part[];     // attention partials of the wavefronts; the sums of A, B, D, E1
    __shared__ __align__(16) float s_q[LR];             // the query: latent part, rotary part
    __shared__ __align__(16) float s_new[LR];           // the new row (last member)
    __shared__ __align__(16) float s_in[128 + R];       // q_nope, q_rope as projected
    __shared__ float s_rope[R + 1];                     // cos, sin of the rotary angles; score of the new token
#if CF_STAMPS
    __shared__ unsigned long long s_ts[kMlaStamps];
    if (threadIdx.x < kMlaStamps) s_ts[threadIdx.x] = 0;
#endif
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, w = blockIdx.x;
    // workgroup w runs on die w % 8; with a multiple of eight heads a head's members share one die, whose L2 then serves
    // the head's weight blocks
    const int head = a.nh % 8 == 0 ? w % 8 + 8 * (w / 8 / TS) : w / TS, j = a.nh % 8 == 0 ? w / 8 % TS : w % TS;
    const int nr = a.n + R, CQq = a.nh * nr, CQ = CQq + LR;
    const bool last = j == TS - 1;
    MLA_STAMP(0);

    // ---- A: projections.  Work item (t, sl): the t-th 128 bytes (eight 16-byte pieces) of the rows of [W_Q | W_KV], row
    //      slice sl of a.ksa <= 4.  A thread owns one piece and eight rows.  (Whole 128-byte lines: with 32-byte tiles of
    //      all rows, which need no slices, the four workgroups of a line hit the same L2 channels with its stride, and
    //      one group in eight was done 2 - 3 us after the others; with 16 slices every reader fetches 16 partial sums.)
    float colsum = 0.f;
    bool mycol = false;
    size_t col = 0;
    unsigned long long launches;
    {
        // tiles of W_Q first, then the nine of W_KV, each matrix with whole tiles of its own
        const int sl = cf::qdiv(w, a.div_t), t = w - sl * a.tiles;
        const bool isq = t < a.tiles - LR / 64;
        const int tk = isq ? t : t - (a.tiles - LR / 64), cols = isq ? CQq : LR;    // tile and width of the matrix
        const int pl = tid & 7, rl = (tid >> 3) * 8;                  // piece of the tile; first of the thread's eight rows of the slice
        const int nrows = sl < a.ksa ? min(a.rows, a.D - sl * a.rows) : 0;          // (rows, D: multiples of eight)
        const uint32_t ld = (uint32_t)cols * 2;
        const Weights W((isq ? a.wq : a.wkv) + (size_t)(sl * a.rows) * cols, (uint32_t)nrows * ld), X(a.x + sl * a.rows, (uint32_t)nrows * 2);
        uint32_t off = 64 * tk + 8 * pl < cols ? (uint32_t)rl * ld + (64 * tk + 8 * pl) * 2 : kNoLoad;
        const h8 xv = X.ld(rl * 2);
        h8 wr[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            wr[k] = W.ld(off);
            off += ld;
        }
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_load_dwordx2 %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)"
                     : "=s"(launches)
                     : "s"(a.counters + (size_t)w * kCounterStride)
                     : "memory");
        if (tid < R / 2) {
            const double inv_freq = exp2(-2.0 * (double)tid / (double)R * a.log2_base);
            cf::rope_cos_sin(a.pos, inv_freq, s_rope[tid], s_rope[R / 2 + tid]);
        }
        float acc[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[c] = 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k)
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[c] = fmaf((float)xv[k], (float)wr[k][c], acc[c]);
        float fold[1];                                                // over the wavefront's rows; a lane keeps column lane / 8
        lanes::fold8<8>(acc, fold);
        s_part[wv * 64 + pl * 8 + (lane >> 3)] = fold[0];
        lds_sync();
        mycol = tid < 64 && sl < a.ksa && 64 * tk + tid < cols;
        col = (size_t)sl * CQ + (isq ? 0 : CQq) + 64 * tk + tid;
        if (mycol)
#pragma unroll
            for (int w8 = 0; w8 < NW; ++w8) colsum += s_part[w8 * 64 + tid];
    }
    const unsigned long long cnt = launches + 1ull;
    const Exchange x = {a.slots, 0, (uint32_t)(cnt + (cnt >> 32)), a.err, a.spin_ticks};
    const __amdgpu_buffer_rsrc_t r = cf::team::slots_rsrc(x);
    if (mycol) cf::team::put(r, a.x1 + col, colsum, x.stamp);
    MLA_STAMP(1);           // A done

    // ---- B: the whole of W_Up[head] (row = nope dimension): thread = 16-byte piece `lane` of the rows wv, wv + 8, ...
    //      The weights do not wait for the query: they are requested behind the put.
    h8 wup[16];
    {
        const Weights W(a.wup + (size_t)head * a.n * L, (uint32_t)a.n * L * 2);
#pragma unroll
        for (int k = 0; k < 16; ++k) wup[k] = W.ld((uint32_t)(wv + 8 * k) * L * 2 + lane * 16);
    }
    // Cached rows of this member.  A row is handled by 16 lanes (a wavefront takes four rows at a time): lane li of a row
    // group owns the latent dimensions 128 k + 8 li .. + 8 (k < 4) and the rotary dimensions 4 li .. + 4, so a row's score
    // needs only the four in-row steps of a cross-lane sum and one exponential serves 36 multiply-adds.  UR rows per row
    // group and batch, two batches in flight; rows past the member's range are zeros and count for nothing.
    constexpr int UR = 4, RPB = NW * 4;                               // rows of the workgroup per step of a batch
    constexpr int step = RPB * UR;
    const int tps = (a.pos + TS - 1) / TS;
    const int t0 = min(j * tps, a.pos), t1 = min(t0 + tps, a.pos);
    const int li = lane & 15, rg = lane >> 4, myrow = wv * 4 + rg;
    h8 kl[2][UR][4];
    h4 kr[2][UR];
    auto request = [&](int buf, int t) {
        __builtin_amdgcn_sched_barrier(0);                            // (behind the last use of the registers)
        const Weights rows(a.cache + (size_t)t * LR, (uint32_t)min(max(t1 - t, 0), step) * LR * 2);
#pragma unroll
        for (int u = 0; u < UR; ++u) {
            const uint32_t off = (uint32_t)(myrow + u * RPB) * LR * 2;
#pragma unroll
            for (int k = 0; k < 4; ++k) kl[buf][u][k] = rows.ld(off + 256 * k + 16 * li);
            kr[buf][u] = __builtin_bit_cast(h4, __builtin_amdgcn_raw_buffer_load_b64(rows.r, off + 2 * L + 8 * li, 0, 0));
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    {
        const int cnt1 = nr + (last ? LR : 0);                        // q of this head; the last member: the new row too
        for (int i = tid; i < cnt1; i += NT) {
            const size_t idx = a.x1 + (i < nr ? head * nr + i : CQq + i - nr);
            pair_t q[kMaxSlices];
            long long tw = 0;
            for (;;) {
#pragma unroll
                for (int k = 0; k < kMaxSlices; ++k) q[k] = cf::team::peek(r, idx + (size_t)min(k, a.ksa - 1) * CQ);
                __builtin_amdgcn_sched_barrier(0);
                bool ok = true;
#pragma unroll
                for (int k = 0; k < kMaxSlices; ++k) ok &= q[k].y == x.stamp;
                if (ok || cf::team::gave_up(x, tw)) break;
            }
            float v = 0.f;
#pragma unroll
            for (int k = 0; k < kMaxSlices; ++k) v += k < a.ksa ? __builtin_bit_cast(float, q[k].x) : 0.f;
            if (i < nr)
                s_in[i < a.n ? i : 128 + i - a.n] = v;
            else
                s_new[i - nr] = v;
        }
    }
    request(0, t0);
    lds_sync();
    MLA_STAMP(2);           // q arrived
    {
        float acc[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[c] = 0.f;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const float qn = s_in[min(wv + 8 * k, a.n - 1)];          // (rows past n carry zero weights)
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[c] = fmaf(qn, (float)wup[k][c], acc[c]);
        }
        float *dst = s_part + wv * L + lane * 8;
        *reinterpret_cast<float4 *>(dst) = make_float4(acc[0], acc[1], acc[2], acc[3]);
        *reinterpret_cast<float4 *>(dst + 4) = make_float4(acc[4], acc[5], acc[6], acc[7]);
        if (tid < R / 2) {                                            // RoPE (pairs d, d + R/2)
            const float c = s_rope[tid], sn = s_rope[R / 2 + tid];
            const float lo = s_in[128 + tid], hi = s_in[128 + tid + R / 2];
            s_q[L + tid] = lo * c - hi * sn;
            s_q[L + tid + R / 2] = hi * c + lo * sn;
            if (last) {
                const float klo = s_new[L + tid], khi = s_new[L + tid + R / 2];
                s_new[L + tid] = klo * c - khi * sn;
                s_new[L + tid + R / 2] = khi * c + klo * sn;
            }
        }
        lds_sync();
        float sum = 0.f;
#pragma unroll
        for (int w8 = 0; w8 < NW; ++w8) sum += s_part[w8 * L + tid];
        s_q[tid] = sum;
        lds_sync();
    }
    request(1, t0 + step);                                            // the registers of W_Up are free
    MLA_STAMP(3);           // query ready
    if (j == 0)                                                       // for cf_mla_debug_export: (q_lat | q_rope) of this head
        for (int i = tid; i < LR; i += NT) a.qdbg[(size_t)head * LR + i] = s_q[i];
    if (last)                                                         // append (Sec. 2.1)
        for (int i = tid; i < LR; i += NT) a.cache[(size_t)a.pos * LR + i] = f2h(s_new[i]);

    // ---- C: attention over the tokens [t0, t1) of this member; the last member also takes the new token
    float ql[4][8], qr4[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int c = 0; c < 8; ++c) ql[k][c] = s_q[128 * k + 8 * li + c] * a.scale_log2e;
#pragma unroll
    for (int c = 0; c < 4; ++c) qr4[c] = s_q[L + 4 * li + c] * a.scale_log2e;
    float m = kNegBig, lsum = 0.f, acc[4][8];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[k][c] = 0.f;
    auto use = [&](int buf, int t) {
        float d[UR];
#pragma unroll
        for (int u = 0; u < UR; ++u) {
            float dd = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int c = 0; c < 8; ++c) dd = fmaf(ql[k][c], (float)kl[buf][u][k][c], dd);
#pragma unroll
            for (int c = 0; c < 4; ++c) dd = fmaf(qr4[c], (float)kr[buf][u][c], dd);
            d[u] = dd;
        }
#pragma unroll
        for (int u = 0; u < UR; ++u) {                                // sum over the 16 lanes of the row
            d[u] = lanes::sum_row(d[u]);
        }
        float mn = m;
#pragma unroll
        for (int u = 0; u < UR; ++u) {
            d[u] = (t + myrow + u * RPB < t1) ? d[u] : kNegBig;
            mn = fmaxf(mn, d[u]);
        }
        const float f = __builtin_amdgcn_exp2f(m - mn);
        m = mn;
        lsum *= f;
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[k][c] *= f;
#pragma unroll
        for (int u = 0; u < UR; ++u) {
            const float pw = (t + myrow + u * RPB < t1) ? __builtin_amdgcn_exp2f(d[u] - mn) : 0.f;
            lsum += pw;
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int c = 0; c < 8; ++c) acc[k][c] = fmaf(pw, (float)kl[buf][u][k][c], acc[k][c]);
        }
    };
    int tt = t0;
    if (t1 > t0) use(0, tt);                                          // (uniform)
    for (; tt + 2 * step < t1; tt += 2 * step) {                      // uniform over the workgroup
        request(0, tt + 2 * step);
        use(1, tt + step);
        request(1, tt + 3 * step);
        use(0, tt + 2 * step);
    }
    // ---- D: the whole of W_Down[head] (row = latent dimension), requested while the last rows are used: thread = 16-byte
    //      piece tid % 16 of the rows tid / 16, + 32, ...
    const int pcD = tid % 16, rowD = tid / 16;
    h8 wdn[16];
    {
        const Weights W(a.wdown + (size_t)head * L * a.v, (uint32_t)L * a.v * 2);
        uint32_t off = 8 * pcD < a.v ? (uint32_t)rowD * a.v * 2 + pcD * 16 : kNoLoad;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            wdn[k] = W.ld(off);
            off += 64 * a.v;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    if (tt + step < t1) use(1, tt + step);
    MLA_STAMP(4);           // rows consumed
    // The four row groups of a wavefront are merged in registers: a swap of half-wavefronts (then of rows of 16 lanes)
    // between two accumulators, followed by an addition, halves their number, so that lane (rg, li) ends with 8 of the 32
    // values of the wavefront.  The eight wavefronts' partials go through LDS (all 32 row groups through LDS, 64 KB written
    // and read back, took 0.5 us more).
    {
        const float mw = lanes::max_groups<16>(m);
        const float f = __builtin_amdgcn_exp2f(m - mw);
        lsum = lanes::sum_groups<16>(lsum * f);
        float h[2][8], q8[8];
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                float p = acc[k][c] * f, q = acc[k + 2][c] * f;
                lanes::swap32(p, q);                                         // lanes 0..31 sum acc[k], lanes 32..63 acc[k + 2]
                h[k][c] = p + q;
            }
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            float p = h[0][c], q = h[1][c];
            lanes::swap16(p, q);                                             // even rows of 16 lanes: h[0], odd rows: h[1]
            q8[c] = p + q;
        }
        // lane (rg, li): latent dimensions 128 (2 (rg >> 1) + (rg & 1)) + 8 li .. + 8 = 128 rg + 8 li
        float *part = s_part + wv * PSTR;
        if (lane == 0) {
            part[0] = mw;
            part[1] = lsum;
        }
        float *dst = part + 4 + 128 * rg + 8 * li;
        *reinterpret_cast<float4 *>(dst) = make_float4(q8[0], q8[1], q8[2], q8[3]);
        *reinterpret_cast<float4 *>(dst + 4) = make_float4(q8[4], q8[5], q8[6], q8[7]);
    }
    if (last && wv == 0) {                                            // score of the new token (its row is not rounded)
        float d = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int c = 0; c < 8; ++c) d = fmaf(ql[k][c], s_new[128 * k + 8 * li + c], d);
#pragma unroll
        for (int c = 0; c < 4; ++c) d = fmaf(qr4[c], s_new[L + 4 * li + c], d);
        d = lanes::sum_row(d);
        if (lane == 0) s_rope[R] = d;
    }
    lds_sync();
    float M, Ls, A = 0.f;
    {
        const int d = tid;                                            // one latent dimension per thread
        M = s_part[0];
#pragma unroll
        for (int w8 = 1; w8 < NW; ++w8) M = fmaxf(M, s_part[w8 * PSTR]);
        if (last) M = fmaxf(M, s_rope[R]);
        Ls = 0.f;
#pragma unroll
        for (int w8 = 0; w8 < NW; ++w8) {
            const float f = __builtin_amdgcn_exp2f(s_part[w8 * PSTR] - M);
            Ls = fmaf(s_part[w8 * PSTR + 1], f, Ls);
            A = fmaf(s_part[w8 * PSTR + 4 + d], f, A);
        }
        if (last) {
            const float f = __builtin_amdgcn_exp2f(s_rope[R] - M);
            Ls += f;
            A = fmaf(s_new[d], f, A);
        }
        s_q[d] = A;                                                   // the merged partial, relative to M (the query is used up)
    }
    lds_sync();
    MLA_STAMP(5);           // C done
    {
        float o[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) o[c] = 0.f;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const float zv = s_q[rowD + 32 * k];
#pragma unroll
            for (int c = 0; c < 8; ++c) o[c] = fmaf(zv, (float)wdn[k][c], o[c]);
        }
        float t[2];
        lanes::fold8<16>(o, t);
        *reinterpret_cast<float2 *>(s_part + wv * 128 + pcD * 8 + 2 * rg) = make_float2(t[0], t[1]);
        lds_sync();
        if (tid < a.v + 2) {
            float sum = 0.f;
            if (tid < a.v) {
#pragma unroll
                for (int w8 = 0; w8 < NW; ++w8) sum += s_part[w8 * 128 + tid];
            }
            cf::team::put(r, a.x3 + ((size_t)head * TS + j) * VS + (tid < a.v ? 2 + tid : tid - a.v), tid < a.v ? sum : tid == a.v ? M : Ls,
                          x.stamp);
        }
    }
    MLA_STAMP(6);           // D done

    // ---- E1: merge of the head's partials, then rows of W_O that belong to this head, column block j of the output: a
    //      partial of out per head
    const int dpE = a.D / 8, pcsE = (dpE + TS - 1) / TS;               // 16-byte pieces of an output row; per member (<= 16)
    const int pcE = tid % 16, rgE = tid / 16, pieceE = j * pcsE + pcE;  // 32 row groups
    const bool liveE = pcE < pcsE && pieceE < dpE;
    h8 wor[4];
    {
        const Weights W(a.wo + (size_t)head * a.v * a.D, (uint32_t)a.v * a.D * 2);
#pragma unroll
        for (int k = 0; k < 4; ++k)                                    // v <= 128: at most four rows per thread
            wor[k] = W.ld(liveE ? (uint32_t)(rgE + 32 * k) * a.D * 2 + pieceE * 16 : kNoLoad);
        __builtin_amdgcn_sched_barrier(0);
    }
    // For cf_mla_debug_export: the member's partial in the latent space, 2 KB on its way while the others' partials arrive.
    // (It costs no time here: without it 22.8 us a step, behind the last poll 22.9, here 22.6 - the polls start a little later
    // and find what they look for.)
    {
        float *dst = a.zpart + ((size_t)head * TS + j) * (L + 2);
        dst[2 + tid] = A;
        if (tid == 0) {
            dst[0] = M;
            dst[1] = Ls;
        }
    }
    {
        // thread = (value c, quarter): four of the 16 partials of value c; every wavefront fetches all maxima and sums
        // (lanes 0..15 and 16..31), so the factors need no barrier
        const int c = min(tid % 128, a.v - 1), qtr = tid / 128;
        const size_t base = a.x3 + (size_t)head * TS * VS;
        pair_t qa[4], qml;
        long long tw = 0;
        for (;;) {
#pragma unroll
            for (int k = 0; k < 4; ++k) qa[k] = cf::team::peek(r, base + (size_t)(4 * qtr + k) * VS + 2 + c);
            qml = cf::team::peek(r, base + (size_t)(lane & 15) * VS + (lane >> 4 & 1));
            __builtin_amdgcn_sched_barrier(0);
            bool ok = qml.y == x.stamp;
#pragma unroll
            for (int k = 0; k < 4; ++k) ok &= qa[k].y == x.stamp;
            if (ok || cf::team::gave_up(x, tw)) break;
        }
        float pm = __builtin_bit_cast(float, qml.x), pl = pm;
        lanes::swap16(pm, pl);                                         // even rows of 16 lanes hold maxima, odd ones sums
        const float Mx = lanes::max_row(pm);
        const float fw = __builtin_amdgcn_exp2f(pm - Mx);              // of partial lane & 15
        const float Lx = lanes::sum_row(pl * fw);
        const int first = __builtin_amdgcn_readfirstlane(4 * qtr);
        float av = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            av = fmaf(__builtin_bit_cast(float, qa[k].x),
                      __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, fw), first + k)), av);
        lds_sync();                                                    // s_part has been read
        s_part[tid] = av / Lx;
    }
    lds_sync();
    MLA_STAMP(7);           // a_head ready
    {
        float o[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) o[c] = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int row = min(rgE + 32 * k, a.v - 1);                // rows past v carry zero weights
            const float av = (s_part[row] + s_part[128 + row]) + (s_part[256 + row] + s_part[384 + row]);
#pragma unroll
            for (int c = 0; c < 8; ++c) o[c] = fmaf(av, (float)wor[k][c], o[c]);
        }
        float t[2];
        lanes::fold8<16>(o, t);
        *reinterpret_cast<float2 *>(s_part + 512 + wv * 128 + pcE * 8 + 2 * rg) = make_float2(t[0], t[1]);
        lds_sync();
        if (tid < 8 * pcsE && j * pcsE * 8 + tid < a.D) {
            float sum = 0.f;
#pragma unroll
            for (int w8 = 0; w8 < NW; ++w8) sum += s_part[512 + w8 * 128 + tid];
            cf::team::put(r, a.x6 + (size_t)head * a.D + j * pcsE * 8 + tid, sum, x.stamp);
        }
    }
    MLA_STAMP(8);           // E1 done

    // ---- E2: sum over the heads (what the paper does with atomicAdd), columns [CW*w, +CW) of the output: thread = (head,
    //      column), one poll each; the heads of a column are added in order by one thread
    {
        const int CW = a.CW;                                           // <= 8
        const int h = cf::qdiv(tid, a.div_cw), c = CW * w + tid - h * CW;
        if (h < a.nh && c < a.D) s_in[tid] = take1(x, r, a.x6 + (size_t)h * a.D + c);
        lds_sync();
        if (h == 0 && c < a.D) {
            float sum = 0.f;
            for (int k = 0; k < a.nh; ++k) sum += s_in[k * CW + tid];
            a.out[c] = f2h(sum);
        }
    }
    if (tid == 0) a.counters[(size_t)w * kCounterStride] = cnt;
    MLA_STAMP(9);
#if CF_STAMPS
    lds_sync();
    if (tid < kMlaStamps && w < 256) g_heads_ts[w * kMlaStamps + tid] = s_ts[tid];
#endif
}

}  // namespace

#if CF_STAMPS
// profiling library only: the stage stamps of the last launch (host buffer of 256 * 16 64-bit words)
extern "C" int cf_mla_heads_trace_read(void *host_dst)
{
    hipError_t e = hipDeviceSynchronize();
    if (e == hipSuccess) e = hipMemcpyFromSymbol(host_dst, HIP_SYMBOL(g_heads_ts), sizeof(unsigned long long) * 256 * kMlaStamps);
    return e == hipSuccess ? CF_OK : CF_EHIP;
}
#endif

namespace cf {
namespace mla {

size_t heads_layout(const cf_mla_config &c, size_t (&first)[3])
{
    first[0] = 0;
    first[1] = first[0] + (size_t)kMaxSlices * (c.n_heads * (c.nope_dim + R) + LR);
    first[2] = first[1] + (size_t)c.n_heads * TS * VS;
    return first[2] + (size_t)c.n_heads * c.d_model;
}

bool slices(const cf_mla_config &c, int *ksa, int *rows)
{
    const int W = c.n_heads * TS, T = (c.n_heads * (c.nope_dim + R) + LR + 63) / 64;
    const int k = W / T < 1 ? 1 : W / T > kMaxSlices ? kMaxSlices : W / T;
    *rows = ((c.d_model + k - 1) / k + 7) / 8 * 8;
    *ksa = (c.d_model + *rows - 1) / *rows;
    return *ksa * T <= W && *rows <= NT;
}

bool heads_prepare()
{
    int per_cu = 0;
    const void *fn = reinterpret_cast<const void *>(fused_mla_heads);
    return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kDynLds) == hipSuccess &&
           hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, NT, kDynLds) == hipSuccess && per_cu >= 1;
}

int heads_launch(const HeadsArgs &a, void *stream)
{
    hipLaunchKernelGGL(fused_mla_heads, dim3(a.W), dim3(NT), kDynLds, static_cast<hipStream_t>(stream), a);
    return (int)hipGetLastError();
}

}  // namespace mla
}  // namespace cf
