// Internal: kernel argument block and launcher interface shared by the host
// side (cf_api.hip) and the device side (cf_fused_kernel.hip) of libcfdecode.
#pragma once

#include "cf_plan_arith.h"

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cf {

constexpr int kThreads = 512;              // threads per workgroup (8 wavefronts of 64)
constexpr int kWaves = kThreads / 64;
constexpr int kOutChunk = 512;             // output columns one wavefront covers with one 128-bit load per lane
constexpr int kP2Stride = 4;               // floats in front of the accumulator in a split-KV partial: m, l, pad, pad
constexpr int kStamps = 24;                // debug time stamps per workgroup
// Bytes between the end of one per-head block of the packed W_qkv and the start of the next.  With
// power-of-two block sizes all workgroups would walk through the memory channels in step (measured:
// a tenth less bandwidth); 256 bytes shift each block by one channel.
constexpr int kQkvBlockPad = 256;
constexpr int kCounterStride = 16;   // 64-bit words between the launch counters of two workgroups (one 128-byte line each)
constexpr int kMaxKSplits = 64;

// Batch tile 16 runs both projections on MFMA tiles; x then sits in LDS as fp16 operands,
// [16][xs16_stride(rows of the longest split)] halves, twice (high parts, low parts of x * gamma).
__host__ __device__ constexpr bool mfma_tiles(int batch_tile) { return batch_tile == 16; }
// (an odd number of 16-byte pieces: the sixteen lanes of an operand read, one per row, then fall into different banks;
// with the 104 pieces of 824 rows and one of padding they met in two)
__host__ __device__ constexpr int xs16_stride(int rps) { return (((rps + 7) >> 3) | 1) << 3; }
// LDS floats that hold x in phase 1.  `layer`: the kernel with RMSNorm; without it head_dim 64 keeps no low parts, which lets it
// take slices of up to 4000 rows (a few shapes with hardly more workgroups than KV heads need more than 2024).
__host__ __device__ constexpr size_t x_lds_floats(int head_dim, int batch_tile, int rps, bool layer)
{
    return mfma_tiles(batch_tile) ? (size_t)(layer || head_dim == 128 ? 16 : 8) * xs16_stride(rps) : (size_t)batch_tile * rps;
}

// The attention output of a head as the operand of the output projection on MFMA tiles: fp16 parts of every value,
// [parts][16][head_dim + kOutPad] halves (rows of an odd number of 16-byte pieces), and two factors per row.  Of a value scaled
// as below, two parts hold 23 bits and three all 24.  Three at head_dim 64, where the vector tile before held fp32; the third costs
// 128 columns 0.1 - 0.5 us (Llama-3-8B shape, 8192 rows, batch 16 107.5 / 107.7 us, Llama-2-7B shape, batch 8 55.4 / 55.9).
constexpr int kOutPad = 8;
__host__ __device__ constexpr int out_parts(int head_dim) { return head_dim == 64 ? 3 : 2; }
__host__ __device__ constexpr int out_operand_floats(int head_dim) { return out_parts(head_dim) * 16 * (head_dim + kOutPad) / 2 + 32; }

constexpr int kFlagPacked = 1;     // weights are in the packed (per-head contiguous) layout of cf_pack_weights
constexpr int kFlagResidual = 2;   // out = x + block output

// Everything the fused kernel needs, passed by value (320 bytes: five 64-byte lines, fetched together at kernel start).  What
// can be computed once per call is computed by the host: a wavefront issues an instruction every four to eight clocks, and
// at small shapes the instructions between two hand-overs are most of the time.
struct LayerPtrs {             // what differs from layer to layer of a stack
    const uint16_t *wqkv, *wo;
    uint16_t *kc, *vc;
    const uint16_t *gamma;     // [D] RMSNorm weight applied to x in front of the projection, or null: x is used as it is
};
struct Params {
    const uint16_t *x;
    const uint16_t *wqkv, *wo; // these five in the order of LayerPtrs: the kernel reads them as one
    uint16_t *kc, *vc;
    const uint16_t *gamma;
    const int32_t *row_pos;    // [B] tokens cached for each batch row (at most pos), or null: pos for every row
    uint16_t *out;
    // workspace
    unsigned long long *done;  // [workgroups][kCounterStride]: launches that workgroup w has completed
    uint32_t *err;         // set to 1 when a spin gave up
    // exchange slots: 64-bit {fp32 bits, launch stamp} pairs
    uint64_t *p1;          // [k_splits][B][Nqkv] partial projections
    uint64_t *p2;          // split-KV partials of head_dim + kP2Stride slots: number (first item of the row) * n_q + head * splits of the
                           // row + split, for the plan's items [B][n_q][kv_splits] (dealt or not, a row has kMaxKvSplits at most, which is
                           // what a handle has room for)
    uint64_t *p3;          // [n_q * row_splits][B][D] per-head partial outputs
    double rope_log2_base; // log2 of the RoPE base: the kernel computes the frequencies base^(-2i/d) itself
    float *dbg_q, *dbg_attn;   // [B][n_q][head_dim] or null
    unsigned long long *dbg_t; // [W][kStamps] wall-clock stamps at phase boundaries, or null
    int D, nq, nkv, B, pos, max_seq, nqkv;
    int W, TS;             // workgroups, workgroups per team (team = one KV head)
    int KS, RPS;           // projection: splits of the reduction dimension, rows of a split (the last one may be shorter)
    int TD;                // attention: tokens of a split are TPS + TD (even split index) or TPS - TD (odd)
    int DSEL;              // TS / KS: selectors advance by this much from one step of a member to the next
    uint32_t div_nkv, div_ks, div_dsel, div_ns;   // for divisions by nkv, KS, DSEL, NS: ceil(2^31 / d)
    int pairmap;           // workgroup -> (team, member) keeps the parity of the workgroup id in the member id
    int NS, TPS;           // attention: splits of the cached sequence, tokens per split
    int NC3, CW3, LRS3;    // output projection: column blocks, columns per block, log2 of the row splits per head
    int CPW;               // output columns a workgroup adds up and writes (an even number)
    uint32_t div_p8;       // the same for RPS / 8
    uint32_t div_n3;       // and for NC3 << LRS3
    // the two layouts of the weights (row-major, packed) as strides in bytes: W_qkv: row, block of head_dim columns; W_o: row,
    // head, chunk of kOutChunk columns
    uint32_t wrow, wblk, orow, ohead, ochunk;
    int flags;             // kFlagPacked, kFlagResidual
    float qk_scale_log2e;  // log2(e)/sqrt(head_dim)
    float eps;             // RMSNorm: added to the mean square
    uint32_t spin_ticks;   // wait limit in 100 MHz ticks (at most 42 s)
    int ragged;            // rows of different lengths, at most one attention item per member: the kernel deals the items itself
    int reserved[9];
};

// A stack of layers in one launch: the pointers of every layer travel by value in the kernel's argument block, behind the
// parameters of the first layer.
constexpr int kMaxStackLayers = 88;        // 320 + 16 + 88 * 40 bytes = 3856 of the 4096 an argument block may have
struct StackArgs {
    Params p;                  // everything of layer 0, and what all layers share
    uint64_t *xslots;          // [B][D / 2] {two fp16 values, stamp}: the hidden state between two layers
    int n_layers, reserved;
    LayerPtrs tab[kMaxStackLayers];
};

// The kernel exists twice: the block alone, and the block with the RMSNorm prologue, the residual epilogue
// and per-row positions
// (a translation unit of its own, compiled from the same source with -DCF_LAYER=1, so that the block kernel
// carries none of that code).
bool wants_layer_kernel(const Params &p);
// Launch the variant for (head_dim, group size, batch tile).  Returns a hipError_t.
hipError_t launch_fused(const Params &p, int head_dim, int group, int batch_tile, size_t lds_bytes,
                        hipStream_t stream);
// The kernel over a.n_layers layers in one launch (a.p must not ask for per-row positions; with RMSNorm or residual the
// slices of the projection have to be multiples of eight rows).
hipError_t launch_fused_stack(const StackArgs &a, int head_dim, int group, int batch_tile, size_t lds_bytes,
                              hipStream_t stream);
// Workgroups of that variant that fit on one CU with `lds_bytes` of LDS each (0 = variant missing).
hipError_t max_workgroups_per_cu(int head_dim, int group, int batch_tile, size_t lds_bytes, bool layer, int *out);
// the same three for the layer kernel (defined by the -DCF_LAYER=1 translation unit; called by those above)
hipError_t launch_layer_stack(const StackArgs &a, int head_dim, int group, int batch_tile, size_t lds_bytes, hipStream_t stream);
hipError_t launch_fused_layer(const Params &p, int head_dim, int group, int batch_tile, size_t lds_bytes,
                              hipStream_t stream);
hipError_t max_workgroups_per_cu_layer(int head_dim, int group, int batch_tile, size_t lds_bytes, int *out);
// LDS floats needed by the three phases for the given plan.
size_t lds_floats(const Params &p, int head_dim, int group, int batch_tile);
// Rearrange row-major weights into the packed layout (see cf_pack_weights in the public header).
hipError_t launch_pack(const uint16_t *wqkv, const uint16_t *wo, uint16_t *wqkv_p, uint16_t *wo_p, int D, int nqkv,
                       int nq, int head_dim, hipStream_t stream);

}  // namespace cf
