// What cf_mla.hip (C ABI, the token-range kernel) and cf_mla_heads.hip (the head-team kernel) share.
#ifndef CF_MLA_INTERNAL_H
#define CF_MLA_INTERNAL_H

#include "../../include/cfdecode.h"

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace cf {
namespace mla {

struct HeadsArgs {
    const uint16_t *x, *wq, *wkv, *wup, *wdown, *wo;
    uint16_t *cache, *out;
    float *qdbg, *zpart;            // for cf_mla_debug_export: [nh][L + R] query (latent | rotated rotary part); [nh][16][2 + L]
                                    // the members' attention partials (maximum, sum, latent vector relative to the maximum)
    uint64_t *slots;
    unsigned long long *counters;
    uint32_t *err;
    size_t x1, x3, x6;              // first slot of each exchange area
    int D, nh, n, v, pos, W;
    int ksa, rows;                  // row slices of the projections, rows per slice (a multiple of eight)
    int tiles, CW;                  // 64-column tiles of W_Q and W_KV, output columns per workgroup
    uint32_t div_t, div_cw;         // ceil(2^31 / d) of both
    float scale_log2e;              // log2(e) / sqrt(nope_dim + rope_dim)
    double log2_base;
    long long spin_ticks;
};

// first slot of the three exchange areas; returns the number of slots in all
size_t heads_layout(const cf_mla_config &c, size_t (&first)[3]);
// row slices of the projections and rows per slice (a multiple of eight, at most 512), such that slices x 64-column tiles
// of [W_Q | W_KV] fit the 16 workgroups per head; false if they do not (no shape cf_mla_create takes)
bool slices(const cf_mla_config &c, int *ksa, int *rows);
// sets the kernel's LDS attribute; false if no workgroup fits a compute unit
bool heads_prepare();
// enqueues the kernel (a.W workgroups); returns the hipError_t of the launch
int heads_launch(const HeadsArgs &a, void *stream);

}  // namespace mla
}  // namespace cf

#endif
