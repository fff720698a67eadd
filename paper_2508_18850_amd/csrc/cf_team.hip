// Team collectives behind the C ABI (cf_team_* in include/cfdecode.h): kernels that run the paper's
// ClusterReduce / ClusterGather schedules (Alg. 1, Alg. 2) among co-resident workgroups through stamped
// exchange slots, one-hop versions of the same collectives, and the two-kernel versions that go through a scratch buffer in global memory instead
// (the "off-chip" column of the paper's Table 1).
#include "../../include/cfdecode.h"
#include "cf_team_device.h"

#include <new>

namespace {

using cf::team::kThreads;
constexpr int kCounterStride = 16;      // 64-bit words between the launch counters of two workgroups
constexpr size_t kMaxElems = 65536;     // largest buffer of one rank (values)

struct TeamArgs {
    const float *in;
    float *out;
    float *scratch;
    uint64_t *slots;                 // [ranks][cap]: pairs of the gather
    uint32_t *boxes;                 // [2][ranks][kMaxRounds][box]: words of the reduce, in two sets
    unsigned long long *counters;    // [ranks][kCounterStride]: launches of the gather, launches of the reduce, boxes and
                                     // words per box the last reduce wrote
    size_t set, box;                 // words of a set, of a box
    uint32_t *err;
    size_t cap, count;
    int N;
    long long spin_ticks;
};

// launch stamp from this workgroup's own launch counter (never 0); the counter is written back at the end
__device__ __forceinline__ uint32_t launch_stamp(const TeamArgs &a, unsigned long long &cnt)
{
    unsigned long long launches;
    asm volatile("s_load_dwordx2 %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)"
                 : "=s"(launches)
                 : "s"(a.counters + (size_t)blockIdx.x * kCounterStride)
                 : "memory");
    cnt = launches + 1ull;
    return (uint32_t)(cnt + (cnt >> 32));
}

// The boxes of this launch of the reduce, and what it owes its predecessor.
struct ReduceLaunch {
    unsigned long long count, wrote;         // launches before this one; what the last one wrote: boxes << 32 | words per box
    cf::team::Boxes x;
    __device__ __forceinline__ explicit ReduceLaunch(const TeamArgs &a)
    {
        asm volatile("s_load_dwordx4 %0, %1, 0x8\n\ts_waitcnt lgkmcnt(0)"
                     : "=s"(state)
                     : "s"(a.counters + (size_t)blockIdx.x * kCounterStride)
                     : "memory");
        count = (unsigned long long)state.y << 32 | state.x;
        wrote = (unsigned long long)state.w << 32 | state.z;
        x.r = __builtin_amdgcn_make_buffer_rsrc(a.boxes + (count & 1 ? a.set : 0), 0, 0xfffffff0u, 0x00020000);
        x.cap = a.box;
        x.err = a.err;
        x.spin_ticks = a.spin_ticks;
    }
    // Of what the last launch wrote in the other set: words from `first` (a multiple of four) up to `end` of this rank's boxes
    // s0 .. s1 - 1 are cleared (no limit: up to what was written)
    static constexpr size_t kAll = ~(size_t)0;
    __device__ __forceinline__ void clear(const TeamArgs &a, int s0, int s1, size_t first, size_t end) const
    {
        const __amdgpu_buffer_rsrc_t other = __builtin_amdgcn_make_buffer_rsrc(a.boxes + (count & 1 ? 0 : a.set), 0, 0xfffffff0u, 0x00020000);
        const cf::team::words4 none = {0u, 0u, 0u, 0u};
        s1 = min(s1, (int)(wrote >> 32));
        end = min(end, (size_t)(uint32_t)wrote);
        for (int s = s0; s < s1; ++s)
            for (size_t i = first + 4 * threadIdx.x; i < end; i += cf::team::kQuads)
                __builtin_amdgcn_raw_buffer_store_b128(none, other, (unsigned)((x.at(blockIdx.x, s) + i) * 4), 0, 16);
    }
    // The count of this launch and what it has written
    __device__ __forceinline__ void finish(const TeamArgs &a, int boxes, size_t words) const
    {
        if (threadIdx.x == 0) {
            unsigned long long *c = a.counters + (size_t)blockIdx.x * kCounterStride;
            c[1] = count + 1;
            c[2] = (unsigned long long)boxes << 32 | (unsigned long long)words;
        }
    }

private:
    cf::team::words4 state;
};

// E 16-byte pieces per thread and chunk; the buffer is worked through chunk by chunk.  32 teams of 8, sum, us a call, with
// 8-byte {value, stamp} pairs / now: one hop, 16384 values 49.9 / 32.9, 16 teams of 16, 3001 values 14.0 / 10.0; rounds, 16 teams of
// 16, 16001 values 100 / 75 (an eighth of that is the emptying of the other set); 1024 values 6.6 - 7, bound by the launch.
template <int E, int OP, bool DIRECT>
__global__ void __launch_bounds__(kThreads) team_reduce_kernel(const TeamArgs a)
{
    using namespace cf::team;
    const int w = blockIdx.x, team = w / a.N, b = w % a.N, tid = threadIdx.x;
    const float *src = a.in + (size_t)w * a.count;
    float *dst = a.out + (size_t)w * a.count;
    f4_t d[E];
    auto load = [&](size_t first) {
#pragma unroll
        for (int e = 0; e < E; ++e) d[e] = load4(src, first + 4 * tid + (size_t)kQuads * e, a.count);
    };
    load(0);
    const ReduceLaunch l(a);
    int boxes = 1;
    // Up to 4096 values in rounds, a box of the other set is cleared between the post of a round and the wait for the peer's:
    // teams of 8, at the end / there, 1 team 1 KB 4.64 / 4.41, 16 KB 7.03 / 6.26, 32 teams 5.03 / 4.80 and 13.2 / 11.35.  At the end
    // with longer buffers (32 teams, 32 KB 15.8 / 17.2, 128 KB 81.0 / 84.3) and with one hop (16 KB 10.2 / 12.2): the stores
    // hold up the polls behind them.
    constexpr bool AMID = !DIRECT && E <= 2;
    size_t first = 0;
    for (; first < a.count; first += (size_t)kQuads * E) {
        if (first) load(first);
        if (DIRECT) {
            post_box<E>(l.x, w, 0, first, a.count, d);
            fold_team<E, OP>(l.x, team * a.N, a.N, b, first, a.count, d);
        } else {
            // Alg. 1: in round s rank b reads what rank b - 2^s holds (its own boxes are all a rank writes)
            int s = 0;
            for (int stride = 1; stride < a.N; stride <<= 1, ++s) {
                post_box<E>(l.x, w, s, first, a.count, d);
                if (AMID) l.clear(a, s, s + 1, first, first + (size_t)kQuads * E);
                fold_box<E, OP>(l.x, team * a.N + (b - stride + a.N) % a.N, s, first, a.count, d);
            }
            boxes = s;
        }
#pragma unroll
        for (int e = 0; e < E; ++e) store4(dst, first + 4 * tid + (size_t)kQuads * e, a.count, d[e]);
    }
    if (AMID) l.clear(a, 0, boxes, first, l.kAll);                // (where the last launch's buffers were the longer ones)
    l.clear(a, AMID ? boxes : 0, kMaxRounds, 0, l.kAll);
    l.finish(a, boxes, a.count);
}

// Two hops with the fewest bytes: rank b folds slice b of the buffer (in rank order) from the others' boxes 0, posts the
// result in box 1, and reads the other slices from their owners.
template <int OP>
__global__ void __launch_bounds__(kThreads) team_reduce_two_hops_kernel(const TeamArgs a)
{
    using namespace cf::team;
    constexpr int C = 8, E = 1;
    const int w = blockIdx.x, team = w / a.N, b = w % a.N;
    const float *src = a.in + (size_t)w * a.count;
    float *dst = a.out + (size_t)w * a.count;
    const size_t t4 = 4 * threadIdx.x;
    const ReduceLaunch l(a);
    const Boxes &x = l.x;
    const unsigned sl = (unsigned)(((a.count + a.N - 1) / a.N + 3) & ~(size_t)3);        // values of a slice: whole pieces
    const size_t lo = min((size_t)b * sl, a.count), hi = min(lo + sl, a.count);
    for (size_t i0 = 0; i0 < a.count; i0 += (size_t)kQuads * C) {          // post what the owners of the other slices need
        f4_t v[C];
#pragma unroll
        for (int k = 0; k < C; ++k) v[k] = load4(src, i0 + t4 + (size_t)kQuads * k, a.count);
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const size_t i = i0 + t4 + (size_t)kQuads * k;
            if (i < a.count && (i < lo || i >= hi)) x.put(x.at(w, 0) + i, v[k]);
        }
    }
    for (size_t first = lo; first < hi; first += (size_t)kQuads * E) {     // fold the own slice, post it
        f4_t d[E];
#pragma unroll
        for (int e = 0; e < E; ++e) d[e] = load4(src, first + t4 + (size_t)kQuads * e, a.count);
        fold_team<E, OP>(x, team * a.N, a.N, b, first, hi, d);
        post_box<E>(x, w, 1, first, hi, d);
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (first + t4 + (size_t)kQuads * e < hi) store4(dst, first + t4 + (size_t)kQuads * e, a.count, d[e]);
    }
    for (size_t i0 = 0; i0 < a.count; i0 += (size_t)kQuads * C) {          // the other slices, from their owners
        words4 q[C];
        long long t0 = 0;
        for (;;) {
            bool ok = true;
#pragma unroll
            for (int k = 0; k < C; ++k) {
                const size_t i = i0 + t4 + (size_t)kQuads * k;
                q[k] = words4{1u, 1u, 1u, 1u};
                if (i < a.count && (i < lo || i >= hi)) q[k] = x.peek(x.at(team * a.N + (int)((unsigned)i / sl), 1) + i);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < C; ++k) ok &= Boxes::there(q[k]);
            if (ok || x.gave_up(t0)) break;
        }
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const size_t i = i0 + t4 + (size_t)kQuads * k;
            if (i < a.count && (i < lo || i >= hi)) store4(dst, i, a.count, Boxes::values(q[k]));
        }
    }
    l.clear(a, 0, kMaxRounds, 0, l.kAll);
    l.finish(a, 2, a.count);
}

// count = values of one segment; a rank's output has N segments
template <bool DIRECT>
__global__ void __launch_bounds__(kThreads) team_gather_kernel(const TeamArgs a)
{
    const int w = blockIdx.x, team = w / a.N, b = w % a.N;
    unsigned long long cnt;
    const cf::team::Exchange x = {a.slots, a.cap, launch_stamp(a, cnt), a.err, a.spin_ticks};
    const float *src = a.in + (size_t)w * a.count;
    float *dst = a.out + (size_t)w * a.count * a.N;
    auto own = [&](size_t i) { return src[i]; };
    auto use = [&](size_t p, float v) { dst[p] = v; };
    if (DIRECT)
        cf::team::gather_direct(x, team * a.N, a.N, b, a.count, own, use);
    else
        cf::team::gather(x, team * a.N, a.N, b, a.count, own, use);
    if (threadIdx.x == 0) a.counters[(size_t)w * kCounterStride] = cnt;
}

// ---- the two-kernel versions: every rank writes its buffer to global memory, the kernel boundary is the
//      synchronisation, then every rank reads what it needs
// (eight independent loads per thread and step, so that these kernels are bound by bandwidth and not by
// one load latency per value)
constexpr int kU = 8;

__global__ void __launch_bounds__(kThreads) team_stage_kernel(const TeamArgs a)
{
    const size_t w = blockIdx.x;
    for (size_t i0 = threadIdx.x; i0 < a.count; i0 += (size_t)kThreads * kU) {
        float v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const size_t i = i0 + (size_t)kThreads * u;
            v[u] = i < a.count ? a.in[w * a.count + i] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const size_t i = i0 + (size_t)kThreads * u;
            if (i < a.count) a.scratch[w * a.count + i] = v[u];
        }
    }
}

template <int OP>
__global__ void __launch_bounds__(kThreads) team_reduce_offchip_kernel(const TeamArgs a)
{
    const int w = blockIdx.x, team = w / a.N;
    for (size_t i0 = threadIdx.x; i0 < a.count; i0 += (size_t)kThreads * kU) {
        float v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const size_t i = i0 + (size_t)kThreads * u;
            v[u] = i < a.count ? a.scratch[(size_t)team * a.N * a.count + i] : 0.f;
        }
        for (int r = 1; r < a.N; ++r) {
            float o[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const size_t i = i0 + (size_t)kThreads * u;
                o[u] = i < a.count ? a.scratch[((size_t)team * a.N + r) * a.count + i] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) v[u] = OP == cf::team::kSum ? v[u] + o[u] : fmaxf(v[u], o[u]);
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const size_t i = i0 + (size_t)kThreads * u;
            if (i < a.count) a.out[(size_t)w * a.count + i] = v[u];
        }
    }
}

__global__ void __launch_bounds__(kThreads) team_gather_offchip_kernel(const TeamArgs a)
{
    const int w = blockIdx.x, team = w / a.N, b = w % a.N;
    for (int j = 0; j < a.N; ++j) {
        const int r = (b - j + a.N) % a.N;
        for (size_t i0 = threadIdx.x; i0 < a.count; i0 += (size_t)kThreads * kU) {
            float v[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const size_t i = i0 + (size_t)kThreads * u;
                v[u] = i < a.count ? a.scratch[((size_t)team * a.N + r) * a.count + i] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const size_t i = i0 + (size_t)kThreads * u;
                if (i < a.count) a.out[((size_t)w * a.N + j) * a.count + i] = v[u];
            }
        }
    }
}

using Kernel = void (*)(const TeamArgs);

template <int OP, bool DIRECT>
Kernel pick_reduce(int e)
{
    switch (e) {
    case 1: return team_reduce_kernel<1, OP, DIRECT>;
    case 2: return team_reduce_kernel<2, OP, DIRECT>;
    }
    return team_reduce_kernel<4, OP, DIRECT>;
}

// 16-byte pieces per thread and chunk: enough for the whole buffer in one chunk up to 4
int pieces_per_thread(size_t values)
{
    return values <= (size_t)cf::team::kQuads ? 1 : values <= (size_t)2 * cf::team::kQuads ? 2 : 4;
}

}  // namespace

struct cf_team_s {
    int max_ranks = 0;
    size_t cap = 0;
    int num_cu = 0;
    char *ws = nullptr;
    size_t head_bytes = 0, slots_bytes = 0, boxes_bytes = 0;     // counters; pairs of the gather; words of the reduce
    size_t box = 0;                         // words of a box
    uint64_t *slots = nullptr;
    uint32_t *boxes = nullptr;
    unsigned long long *counters = nullptr;
    uint32_t *err = nullptr;
    float *scratch = nullptr;
    long long spin_ticks = 200000000LL;     // 2 s
    int last_ranks = 0;                     // workgroups of the previous launch
    int last_hip = 0;
};

namespace {

int fail(cf_team t, hipError_t e)
{
    if (t) t->last_hip = (int)e;
    return CF_EHIP;
}

bool pow2(int v) { return v > 0 && (v & (v - 1)) == 0; }

int check_call(cf_team t, int32_t teams, int32_t team_size, const void *in, const void *out, size_t elems, int32_t mode)
{
    if (mode != CF_TEAM_ROUNDS && mode != CF_TEAM_TWO_KERNELS && mode != CF_TEAM_DIRECT && mode != CF_TEAM_TWO_HOPS)
        return CF_EINVAL;
    if (!t || !in || !out || teams < 1 || !pow2(team_size) || team_size > 16 || elems < 1) return CF_EINVAL;
    if ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) & 3u) return CF_EINVAL;
    if ((long)teams * team_size > t->max_ranks) return CF_EINVAL;
    // receivers spin: all workgroups of the launch must be resident, one per compute unit
    if ((long)teams * team_size > t->num_cu) return CF_EUNSUPPORTED;
    return CF_OK;
}

// Counters, pairs and boxes cleared.
hipError_t reset(cf_team t)
{
    const hipError_t e = hipMemset(t->ws, 0, t->head_bytes + t->slots_bytes + t->boxes_bytes);
    return e == hipSuccess ? hipDeviceSynchronize() : e;
}

// Every workgroup counts its own launches and all of a launch must agree on the count: when the number of
// workgroups changes, the counts (and with them all stamps) start together again.
int same_grid(cf_team t, int ranks)
{
    if (ranks == t->last_ranks) return CF_OK;
    hipError_t e = hipDeviceSynchronize();
    if (e == hipSuccess) e = reset(t);
    if (e != hipSuccess) return fail(t, e);
    t->last_ranks = ranks;
    return CF_OK;
}

TeamArgs make_args(cf_team t, const float *in, float *out, size_t count, int n)
{
    TeamArgs a;
    a.in = in;
    a.out = out;
    a.scratch = t->scratch;
    a.slots = t->slots;
    a.boxes = t->boxes;
    a.set = (size_t)t->max_ranks * cf::team::kMaxRounds * t->box;
    a.box = t->box;
    a.counters = t->counters;
    a.err = t->err;
    a.cap = t->cap;
    a.count = count;
    a.N = n;
    a.spin_ticks = t->spin_ticks;
    return a;
}

}  // namespace

extern "C" {

int cf_team_create(int32_t max_ranks, size_t max_elems, cf_team *out)
{
    if (!out || max_ranks < 1 || max_elems < 1 || max_elems > kMaxElems) return CF_EINVAL;
    *out = nullptr;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    hipDeviceProp_t prop;
    if (e == hipSuccess) e = hipGetDeviceProperties(&prop, dev);
    if (e != hipSuccess) return CF_EHIP;
    cf_team t = new (std::nothrow) cf_team_s();
    if (!t) return CF_ENOMEM;
    t->max_ranks = max_ranks;
    t->cap = max_elems;
    t->num_cu = prop.multiProcessorCount;
    const size_t head = 256 + (size_t)max_ranks * kCounterStride * sizeof(unsigned long long);
    // (what the exchange area of a handle took before there were two sets of words: the limit of a handle stays)
    if ((size_t)max_ranks * cf::team::kMaxRounds * max_elems * sizeof(uint64_t) > 0xfffffff0ull) {
        delete t;
        return CF_EUNSUPPORTED;
    }
    auto up = [](size_t v) { return (v + 255) / 256 * 256; };
    t->head_bytes = up(head);
    t->slots_bytes = up((size_t)max_ranks * max_elems * sizeof(uint64_t));
    t->box = (max_elems + 3) & ~(size_t)3;
    t->boxes_bytes = (size_t)2 * max_ranks * cf::team::kMaxRounds * t->box * sizeof(uint32_t);       // (a set: 32-bit byte offsets)
    const size_t scratch_bytes = (size_t)max_ranks * max_elems * sizeof(float);
    e = hipMalloc(reinterpret_cast<void **>(&t->ws), t->head_bytes + t->slots_bytes + t->boxes_bytes + scratch_bytes);
    if (e != hipSuccess) {
        delete t;
        return e == hipErrorOutOfMemory ? CF_ENOMEM : CF_EHIP;
    }
    t->err = reinterpret_cast<uint32_t *>(t->ws + 128);
    t->counters = reinterpret_cast<unsigned long long *>(t->ws + 256);
    t->slots = reinterpret_cast<uint64_t *>(t->ws + t->head_bytes);
    t->boxes = reinterpret_cast<uint32_t *>(t->ws + t->head_bytes + t->slots_bytes);
    t->scratch = reinterpret_cast<float *>(t->ws + t->head_bytes + t->slots_bytes + t->boxes_bytes);
    e = reset(t);
    if (e != hipSuccess) {
        (void)hipFree(t->ws);
        delete t;
        return CF_EHIP;
    }
    *out = t;
    return CF_OK;
}

int cf_team_destroy(cf_team t)
{
    if (!t) return CF_EINVAL;
    hipError_t e = hipFree(t->ws);
    delete t;
    return e == hipSuccess ? CF_OK : CF_EHIP;
}

int cf_team_reduce(cf_team t, int32_t teams, int32_t team_size, int32_t op, const float *in, float *out, size_t elems,
                   int32_t mode, void *stream)
{
    int rc = check_call(t, teams, team_size, in, out, elems, mode);
    if (rc != CF_OK) return rc;
    if ((op != CF_TEAM_SUM && op != CF_TEAM_MAX) || elems > t->cap) return CF_EINVAL;
    if (mode != CF_TEAM_TWO_KERNELS && (rc = same_grid(t, teams * team_size)) != CF_OK) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const TeamArgs a = make_args(t, in, out, elems, team_size);
    const dim3 grid(teams * team_size), block(kThreads);
    if (mode == CF_TEAM_TWO_KERNELS) {
        hipLaunchKernelGGL(team_stage_kernel, grid, block, 0, s, a);
        if (op == CF_TEAM_SUM)
            hipLaunchKernelGGL(team_reduce_offchip_kernel<cf::team::kSum>, grid, block, 0, s, a);
        else
            hipLaunchKernelGGL(team_reduce_offchip_kernel<cf::team::kMax>, grid, block, 0, s, a);
    } else {
        const int e = pieces_per_thread(elems);
        Kernel k;
        if (mode == CF_TEAM_TWO_HOPS)
            k = op == CF_TEAM_SUM ? team_reduce_two_hops_kernel<cf::team::kSum> : team_reduce_two_hops_kernel<cf::team::kMax>;
        else if (mode == CF_TEAM_DIRECT)
            k = op == CF_TEAM_SUM ? pick_reduce<cf::team::kSum, true>(e) : pick_reduce<cf::team::kMax, true>(e);
        else
            k = op == CF_TEAM_SUM ? pick_reduce<cf::team::kSum, false>(e) : pick_reduce<cf::team::kMax, false>(e);
        hipLaunchKernelGGL(k, grid, block, 0, s, a);
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? CF_OK : fail(t, e);
}

int cf_team_gather(cf_team t, int32_t teams, int32_t team_size, const float *in, float *out, size_t elems,
                   int32_t mode, void *stream)
{
    int rc = check_call(t, teams, team_size, in, out, elems, mode);
    if (rc != CF_OK) return rc;
    if (elems * (size_t)team_size > t->cap || mode == CF_TEAM_TWO_HOPS) return CF_EINVAL;
    if (mode != CF_TEAM_TWO_KERNELS && (rc = same_grid(t, teams * team_size)) != CF_OK) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const TeamArgs a = make_args(t, in, out, elems, team_size);
    const dim3 grid(teams * team_size), block(kThreads);
    if (mode == CF_TEAM_TWO_KERNELS) {
        hipLaunchKernelGGL(team_stage_kernel, grid, block, 0, s, a);
        hipLaunchKernelGGL(team_gather_offchip_kernel, grid, block, 0, s, a);
    } else if (mode == CF_TEAM_DIRECT) {
        hipLaunchKernelGGL(team_gather_kernel<true>, grid, block, 0, s, a);
    } else {
        hipLaunchKernelGGL(team_gather_kernel<false>, grid, block, 0, s, a);
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? CF_OK : fail(t, e);
}

int cf_team_status(cf_team t, void *stream)
{
    if (!t) return CF_EINVAL;
    hipError_t e = hipStreamSynchronize(static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail(t, e);
    uint32_t flag = 0;
    e = hipMemcpy(&flag, t->err, sizeof flag, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return fail(t, e);
    if (flag) {
        e = reset(t);                                // launch counters, stamps and boxes start afresh
        if (e != hipSuccess) return fail(t, e);
        return CF_ETIMEOUT;
    }
    return CF_OK;
}

int cf_team_set_spin_limit(cf_team t, int32_t spin_limit_us)
{
    if (!t || spin_limit_us < 0) return CF_EINVAL;
    t->spin_ticks = (long long)spin_limit_us * 100;
    return CF_OK;
}

}  // extern "C"
