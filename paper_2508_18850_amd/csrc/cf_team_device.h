// Team collectives for gfx950: what a group of co-resident workgroups can do in place of the paper's
// ClusterReduce (Alg. 1) and ClusterGather (Alg. 2), which run over the distributed shared memory of a
// thread-block cluster.  CDNA4 has no such memory; the nearest thing is an exchange through global
// memory that never leaves the kernel: every fp32 value travels as a 64-bit {value, stamp} pair written
// with one write-through store and polled by the receiver until the stamp is the current one.  No flag,
// no fence, no atomic; a value is either the old pair or the new one.
//
// The all-reduce of whole buffers (cf_team_reduce) needs no stamps: see "four bytes per value" below.
//
// Two schedules.  The paper's: log2(N) rounds, in round s rank b sends to rank (b + 2^s) mod N and
// receives from rank (b - 2^s) mod N.  And a direct one: every rank posts its data once and reads the
// posts of its N - 1 peers, one hop in place of log2(N); a hop through memory costs microseconds here
// where a hop through a cluster's shared memory costs a fraction of one, so the direct schedule is the one
// the fused decode kernel uses.
//
// Buffers are worked through in chunks (E values or 16-byte pieces per thread in registers), so that the register use does
// not grow with the buffer.
//
// These are device functions to be called by all threads of a workgroup; every workgroup of the team
// must be resident at the same time (the caller's launch has to guarantee that), because receivers spin.
#ifndef CF_TEAM_DEVICE_H
#define CF_TEAM_DEVICE_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cf {
namespace team {

typedef uint32_t pair_t __attribute__((ext_vector_type(2)));

constexpr int kThreads = 512;      // threads per workgroup the functions are written for
constexpr int kMaxRounds = 4;      // N <= 16

enum Op { kSum = 0, kMax = 1 };

// Exchange area of one launch: rank r's slots = slots[r * kMaxRounds * cap ...] for the two-hop reduce of pairs,
// slots[r * cap ...] for the gather (cap in pairs).
struct Exchange {
    uint64_t *slots;     // device memory, cleared once when it is allocated
    size_t cap;          // pairs per inbox
    uint32_t stamp;      // stamp of this launch, never 0
    uint32_t *err;       // set to 1 when a wait gave up
    long long spin_ticks;    // give up after this many ticks of the 100 MHz wall clock (0: at the first failed look)
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t slots_rsrc(const Exchange &x)
{
    return __builtin_amdgcn_make_buffer_rsrc(x.slots, 0, 0xfffffff8u, 0x00020000);
}

__device__ __forceinline__ void put(__amdgpu_buffer_rsrc_t r, size_t idx, float v, uint32_t stamp)
{
    pair_t d = {__builtin_bit_cast(uint32_t, v), stamp};
    __builtin_amdgcn_raw_buffer_store_b64(d, r, (unsigned)(idx * 8), 0, 16);      // sc1: through to memory
}

__device__ __forceinline__ pair_t peek(__amdgpu_buffer_rsrc_t r, size_t idx)
{
    return __builtin_amdgcn_raw_buffer_load_b64(r, (unsigned)(idx * 8), 0, 16);   // sc1: not from a stale cache
}

// true when the caller should stop waiting (the error flag is set then)
__device__ __forceinline__ bool gave_up(const Exchange &x, long long &t0)
{
    __builtin_amdgcn_s_sleep(1);
    const long long now = wall_clock64();
    if (t0 == 0) t0 = now;
    if (now - t0 >= x.spin_ticks) {                 // a limit of 0 gives up at the first failed look
        __hip_atomic_store(x.err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return true;
    }
    return false;
}

constexpr int kPolls = 32;         // polls a thread keeps in flight: the receive rate is kPolls x 8 bytes per round trip

template <int OP>
__device__ __forceinline__ float fold(float a, float b)
{
    return OP == kSum ? a + b : fmaxf(a, b);
}

// Fold what the N ranks of a team have posted at positions first + tid + kThreads*e (< end) of the area that
// starts `area` pairs into every rank's slots, in rank order, the rank's own values d[] at their place.
template <int E, int OP>
__device__ __forceinline__ void fold_posts(const Exchange &x, __amdgpu_buffer_rsrc_t r, int team_first_rank, int N, int b,
                                           size_t area, size_t first, size_t end, float (&d)[E])
{
    const size_t tid = threadIdx.x;
    const size_t box = (size_t)kMaxRounds * x.cap;                    // a rank's whole slot area
    constexpr int P = E >= kPolls ? 1 : kPolls / E;                   // peers polled together
    float acc[E];
    for (int r0 = 0; r0 < N; r0 += P) {
        pair_t q[P][E];
        long long t0 = 0;
        for (;;) {
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const int peer = r0 + p;
#pragma unroll
                for (int e = 0; e < E; ++e) q[p][e] = pair_t{0u, x.stamp};
                if (peer < N && peer != b) {                          // uniform over the workgroup
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        const size_t i = first + tid + (size_t)kThreads * e;
                        q[p][e] = peek(r, (size_t)(team_first_rank + peer) * box + area + (i < end ? i : first));
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            bool ok = true;
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const size_t i = first + tid + (size_t)kThreads * e;
                    ok &= (i >= end) | (q[p][e].y == x.stamp);
                }
            if (ok || gave_up(x, t0)) break;
        }
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int peer = r0 + p;
            if (peer < N) {
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const float v = peer == b ? d[e] : __builtin_bit_cast(float, q[p][e].x);
                    acc[e] = peer == 0 ? v : fold<OP>(acc[e], v);
                }
            }
        }
    }
#pragma unroll
    for (int e = 0; e < E; ++e) d[e] = acc[e];
}

// The all-reduce in two hops with the fewest bytes: rank b folds slice b of the buffer (count / N values, in
// rank order) from the posts of the others, posts the result, and reads the other slices from their owners.
// A rank receives 2 * (N - 1) / N * count values, against (N - 1) * count in one hop.  own(i) gives value i of
// the rank's buffer, use(i, v) receives value i of the result.
template <int OP, class Own, class Use>
__device__ __forceinline__ void reduce_two_hops(const Exchange &x, int team_first_rank, int N, int b, size_t count,
                                                Own &&own, Use &&use)
{
    constexpr int C = 16, E = 4;
    const __amdgpu_buffer_rsrc_t r = slots_rsrc(x);
    const size_t tid = threadIdx.x;
    const size_t box = (size_t)kMaxRounds * x.cap;
    const size_t mine = (size_t)(team_first_rank + b) * box;
    const unsigned sl = (unsigned)((count + N - 1) / N);              // values of a slice; count <= cap < 2^32
    const size_t lo = (size_t)b * sl < count ? (size_t)b * sl : count;
    const size_t hi = lo + sl < count ? lo + sl : count;
    for (size_t i0 = 0; i0 < count; i0 += (size_t)kThreads * C) {     // post what the owners of the other slices need
        float v[C];
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const size_t i = i0 + tid + (size_t)kThreads * k;
            v[k] = i < count ? own(i) : 0.f;
        }
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const size_t i = i0 + tid + (size_t)kThreads * k;
            if (i < count && (i < lo || i >= hi)) put(r, mine + i, v[k], x.stamp);
        }
    }
    for (size_t first = lo; first < hi; first += (size_t)kThreads * E) {      // fold the own slice, post it
        float d[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const size_t i = first + tid + (size_t)kThreads * e;
            d[e] = i < hi ? own(i) : 0.f;
        }
        fold_posts<E, OP>(x, r, team_first_rank, N, b, 0, first, hi, d);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const size_t i = first + tid + (size_t)kThreads * e;
            if (i < hi) {
                put(r, mine + x.cap + i, d[e], x.stamp);              // second area of the rank's slots
                use(i, d[e]);
            }
        }
    }
    for (size_t i0 = 0; i0 < count; i0 += (size_t)kThreads * C) {     // the other slices, from their owners
        pair_t q[C];
        long long t0 = 0;
        for (;;) {
#pragma unroll
            for (int k = 0; k < C; ++k) {
                const size_t i = i0 + tid + (size_t)kThreads * k;
                const bool want = i < count && (i < lo || i >= hi);
                const unsigned owner = (unsigned)i / sl;
                q[k] = want ? peek(r, (size_t)(team_first_rank + owner) * box + x.cap + i) : pair_t{0u, x.stamp};
            }
            __builtin_amdgcn_sched_barrier(0);
            bool ok = true;
#pragma unroll
            for (int k = 0; k < C; ++k) ok &= q[k].y == x.stamp;
            if (ok || gave_up(x, t0)) break;
        }
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const size_t i = i0 + tid + (size_t)kThreads * k;
            if (i < count && (i < lo || i >= hi)) use(i, __builtin_bit_cast(float, q[k].x));
        }
    }
}

// ---- all-reduce of whole buffers, four bytes per value ---------------------------------------------------------------
//
// The stamp of a pair doubles the bytes, and a pair is eight bytes at most: a rank's receive rate was that of 8-byte polls
// (some 30 GB/s per workgroup).  Here a posted value is its own arrival mark: an empty box holds zeros, a value's bits are sent
// inverted and are there as soon as the word is not zero, and four words go in one 16-byte access, of which each is judged by
// itself.  There are two sets of boxes, used by launches in turn; a launch clears what its predecessor has written in the
// other set (nobody reads that any more: launches on one handle follow each other), so that the set is empty when the
// next launch takes it.  A value with all bits set, a NaN, is sent as the NaN next to it.
typedef uint32_t words4 __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef float f4u_t __attribute__((ext_vector_type(4), aligned(4)));      // user buffers are 4-byte aligned

constexpr int kQuads = kThreads * 4;       // values a workgroup handles with one 16-byte access per thread

// Box s of rank r in the set of this launch = words[(r * kMaxRounds + s) * cap ...], cap a multiple of four.
struct Boxes {
    __amdgpu_buffer_rsrc_t r;
    size_t cap;
    uint32_t *err;
    long long spin_ticks;
    __device__ __forceinline__ size_t at(int rank, int s) const { return ((size_t)rank * kMaxRounds + s) * cap; }
    __device__ __forceinline__ void put(size_t idx, const f4_t &v) const
    {
        words4 q = ~__builtin_bit_cast(words4, v);
#pragma unroll
        for (int k = 0; k < 4; ++k) q[k] = max(q[k], 1u);
        __builtin_amdgcn_raw_buffer_store_b128(q, r, (unsigned)(idx * 4), 0, 16);                    // sc1: through to memory
    }
    __device__ __forceinline__ words4 peek(size_t idx) const
    {
        return __builtin_amdgcn_raw_buffer_load_b128(r, (unsigned)(idx * 4), 0, 16);                 // sc1: not from a stale cache
    }
    static __device__ __forceinline__ bool there(const words4 &q)
    {
        return (q.x != 0u) & (q.y != 0u) & (q.z != 0u) & (q.w != 0u);
    }
    static __device__ __forceinline__ f4_t values(const words4 &q) { return __builtin_bit_cast(f4_t, ~q); }
    __device__ __forceinline__ bool gave_up(long long &t0) const
    {
        return team::gave_up(Exchange{nullptr, 0, 0, err, spin_ticks}, t0);
    }
};

// Values i .. i + 3 of a user buffer of `count` values (zeros past its end), and the same stored.
__device__ __forceinline__ f4_t load4(const float *src, size_t i, size_t count)
{
    if (i + 4 <= count) return *reinterpret_cast<const f4u_t *>(src + i);
    f4_t v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 3; ++k)
        if (i + k < count) v[k] = src[i + k];
    return v;
}
__device__ __forceinline__ void store4(float *dst, size_t i, size_t count, const f4_t &v)
{
    if (i + 4 <= count) {
        *reinterpret_cast<f4u_t *>(dst + i) = v;
        return;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k)
        if (i + k < count) dst[i + k] = v[k];
}

template <int OP>
__device__ __forceinline__ f4_t fold4(const f4_t &a, const f4_t &b)
{
    f4_t v;
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = fold<OP>(a[k], b[k]);
    return v;
}

// Wait for box s of rank `from`, values first + 4 tid + kQuads e (e < E, < count), and fold them into d (Alg. 1: D_b op B_b).
template <int E, int OP>
__device__ __forceinline__ void fold_box(const Boxes &x, int from, int s, size_t first, size_t count, f4_t (&d)[E])
{
    const size_t base = x.at(from, s), i0 = first + 4 * threadIdx.x;
    words4 q[E];
    long long t0 = 0;
    for (;;) {
        bool ok = true;
#pragma unroll
        for (int e = 0; e < E; ++e) q[e] = x.peek(base + (i0 + (size_t)kQuads * e < count ? i0 + (size_t)kQuads * e : 0));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < E; ++e) ok &= (i0 + (size_t)kQuads * e >= count) | Boxes::there(q[e]);
        if (ok || x.gave_up(t0)) break;
    }
#pragma unroll
    for (int e = 0; e < E; ++e) d[e] = fold4<OP>(d[e], Boxes::values(q[e]));
}

// d = fold, in rank order, of box 0 of the N ranks of the team at the same values (own d at its place); kInFlight 16-byte
// polls per thread go out before the first one is looked at.
template <int E, int OP>
__device__ __forceinline__ void fold_team(const Boxes &x, int team_first_rank, int N, int b, size_t first, size_t count, f4_t (&d)[E])
{
    constexpr int kInFlight = 16, P = kInFlight / E;                  // peers polled together
    const size_t i0 = first + 4 * threadIdx.x;
    f4_t acc[E];
    for (int r0 = 0; r0 < N; r0 += P) {
        words4 q[P][E];
        long long t0 = 0;
        for (;;) {
            bool ok = true;
#pragma unroll
            for (int p = 0; p < P; ++p)
                if (r0 + p < N && r0 + p != b)                        // (uniform)
#pragma unroll
                    for (int e = 0; e < E; ++e)
                        q[p][e] = x.peek(x.at(team_first_rank + r0 + p, 0) + (i0 + (size_t)kQuads * e < count ? i0 + (size_t)kQuads * e : first));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int p = 0; p < P; ++p)
                if (r0 + p < N && r0 + p != b)
#pragma unroll
                    for (int e = 0; e < E; ++e) ok &= (i0 + (size_t)kQuads * e >= count) | Boxes::there(q[p][e]);
            if (ok || x.gave_up(t0)) break;
        }
#pragma unroll
        for (int p = 0; p < P; ++p)
            if (r0 + p < N)
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const f4_t v = r0 + p == b ? d[e] : Boxes::values(q[p][e]);
                    acc[e] = r0 + p == 0 ? v : fold4<OP>(acc[e], v);
                }
    }
#pragma unroll
    for (int e = 0; e < E; ++e) d[e] = acc[e];
}

template <int E>
__device__ __forceinline__ void post_box(const Boxes &x, int rank, int s, size_t first, size_t count, const f4_t (&d)[E])
{
    const size_t base = x.at(rank, s), i0 = first + 4 * threadIdx.x;
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (i0 + (size_t)kQuads * e < count) x.put(base + i0 + (size_t)kQuads * e, d[e]);
}

constexpr int kGatherBatch = 16;   // values per thread and step of the gathers

// Alg. 2: all-gather.  A rank's buffer has N segments of `seg` values; own(i) gives value i < seg of the
// rank's own data; use(p, v) receives value p of the gathered buffer, p in [0, N*seg), where segment j is the
// data of rank (b - j) mod N.  Nothing is held in registers between the rounds: what arrived in the rank's
// inbox in the earlier rounds is read there again when it is passed on.
template <class Own, class Use>
__device__ __forceinline__ void gather(const Exchange &x, int team_first_rank, int N, int b, size_t seg, Own &&own, Use &&use)
{
    constexpr int C = kGatherBatch;
    const __amdgpu_buffer_rsrc_t r = slots_rsrc(x);
    const size_t tid = threadIdx.x;
    const size_t inbox = (size_t)(team_first_rank + b) * x.cap;
    // wait for positions i0 + tid + kThreads*k of the inbox that are in [seg, end); positions below seg are the rank's own
    auto fetch = [&](size_t i0, size_t end, float (&v)[C]) {
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const size_t i = i0 + tid + (size_t)kThreads * k;
            v[k] = i < seg ? own(i) : 0.f;
        }
        if (i0 + (size_t)kThreads * C <= seg) return;                 // the whole step is own data (uniform)
        pair_t q[C];
        long long t0 = 0;
        for (;;) {
#pragma unroll
            for (int k = 0; k < C; ++k) {
                const size_t i = i0 + tid + (size_t)kThreads * k;
                q[k] = peek(r, inbox + (i >= seg && i < end ? i : seg));
            }
            __builtin_amdgcn_sched_barrier(0);
            bool ok = true;
#pragma unroll
            for (int k = 0; k < C; ++k) {
                const size_t i = i0 + tid + (size_t)kThreads * k;
                ok &= (i < seg) | (i >= end) | (q[k].y == x.stamp);
            }
            if (ok || gave_up(x, t0)) break;
        }
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const size_t i = i0 + tid + (size_t)kThreads * k;
            if (i >= seg) v[k] = __builtin_bit_cast(float, q[k].x);
        }
    };
    for (int stride = 1; stride < N; stride <<= 1) {
        const int to = (b + stride) % N;
        const size_t have = seg * (size_t)stride;                     // values this rank holds so far
        const size_t outbox = (size_t)(team_first_rank + to) * x.cap + have;    // they become the peer's next segments
        for (size_t i0 = 0; i0 < have; i0 += (size_t)kThreads * C) {
            float v[C];
            fetch(i0, have, v);
#pragma unroll
            for (int k = 0; k < C; ++k) {
                const size_t i = i0 + tid + (size_t)kThreads * k;
                if (i < have) put(r, outbox + i, v[k], x.stamp);
            }
        }
    }
    const size_t all = seg * (size_t)N;
    for (size_t i0 = 0; i0 < all; i0 += (size_t)kThreads * C) {
        float v[C];
        fetch(i0, all, v);
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const size_t i = i0 + tid + (size_t)kThreads * k;
            if (i < all) use(i, v[k]);
        }
    }
}

// The same result in one hop: every rank posts its segment in its own outbox and reads the N - 1 others.
template <class Own, class Use>
__device__ __forceinline__ void gather_direct(const Exchange &x, int team_first_rank, int N, int b, size_t seg, Own &&own,
                                              Use &&use)
{
    constexpr int C = kGatherBatch;
    const __amdgpu_buffer_rsrc_t r = slots_rsrc(x);
    const size_t tid = threadIdx.x;
    for (size_t i0 = 0; i0 < seg; i0 += (size_t)kThreads * C) {
        float v[C];
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const size_t i = i0 + tid + (size_t)kThreads * k;
            v[k] = i < seg ? own(i) : 0.f;
        }
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const size_t i = i0 + tid + (size_t)kThreads * k;
            if (i < seg) {
                put(r, (size_t)(team_first_rank + b) * x.cap + i, v[k], x.stamp);
                use(i, v[k]);
            }
        }
    }
    // positions seg .. N*seg of the result, as one index space: position p is value p % seg of rank (b - p / seg) mod N
    const size_t all = seg * (size_t)N;
    for (size_t i0 = seg; i0 < all; i0 += (size_t)kThreads * C) {
        pair_t q[C];
        long long t0 = 0;
        for (;;) {
#pragma unroll
            for (int k = 0; k < C; ++k) {
                const size_t i = i0 + tid + (size_t)kThreads * k;
                const unsigned p = (unsigned)(i < all ? i : seg);      // all <= cap < 2^32
                const unsigned j = p / (unsigned)seg;
                q[k] = peek(r, (size_t)(team_first_rank + (b - (int)j + N) % N) * x.cap + (p - j * (unsigned)seg));
            }
            __builtin_amdgcn_sched_barrier(0);
            bool ok = true;
#pragma unroll
            for (int k = 0; k < C; ++k) {
                const size_t i = i0 + tid + (size_t)kThreads * k;
                ok &= (i >= all) | (q[k].y == x.stamp);
            }
            if (ok || gave_up(x, t0)) break;
        }
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const size_t i = i0 + tid + (size_t)kThreads * k;
            if (i < all) use(i, __builtin_bit_cast(float, q[k].x));
        }
    }
}

}  // namespace team
}  // namespace cf
#endif
