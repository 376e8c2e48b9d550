// kernels.h -- host launchers of the gfx950 kernels (all asynchronous on the
// given stream; they return the launch error, if any).
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <utility>

#include "common.h"

namespace msi {

// Per-launch telemetry: while `stop` is set, kernels launched through
// launch_k carry HIP events that the runtime records at the first kernel's
// start and at each kernel's end (the last one's end is the one that stays),
// so the measured span is the kernels' own execution, not the host's
// enqueue gaps.
struct LaunchTiming {
    hipEvent_t start = nullptr, stop = nullptr;
};
inline LaunchTiming &launch_timing()
{
    static thread_local LaunchTiming t;
    return t;
}

template <typename... KArgs, typename... Args>
inline void launch_k(void (*k)(KArgs...), dim3 grid, dim3 block, size_t lds, hipStream_t s, Args &&...args)
{
    LaunchTiming &t = launch_timing();
    if (t.stop) {
        hipExtLaunchKernelGGL<KArgs...>(k, grid, block, uint32_t(lds), s, t.start, t.stop, 0u,
                                        static_cast<KArgs>(std::forward<Args>(args))...);
        t.start = nullptr;
    } else {
        k<<<grid, block, lds, s>>>(std::forward<Args>(args)...);
    }
}

// ---- router and permutation (route.hip)
hipError_t launch_router_logits_f32(const float *x, const float *wr, const float *bias, float *L, int T, int d,
                                    int E, hipStream_t s);
hipError_t launch_router_logits_bf16(const uint16_t *x, const uint16_t *wr, const float *bias, float *L, int T,
                                     int d, int E, hipStream_t s);
// raise the dynamic LDS limit of the kernels that use more than 64 KiB
hipError_t init_kernel_attributes();

// Let kernel f use all of the CU's 160 KiB of LDS (dynamic part = 160 KiB
// minus its static LDS).
inline hipError_t allow_large_lds(const void *f)
{
    hipFuncAttributes a{};
    hipError_t e = hipFuncGetAttributes(&a, f);
    if (e != hipSuccess)
        return e;
    return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                               int(160 * 1024 - a.sharedSizeBytes));
}
// Outputs of one routing (device arrays, see msi_routing).
struct RouteOut {
    int32_t *idx;
    float *w;
    int32_t *counts;
    int32_t *offsets;
    int32_t *demand;
    int32_t *perm;
    int32_t *inv;
    float *row_weight;
};
// top-K + restricted softmax + permutation of logits L (bias included): one
// fused workgroup when T <= 16, else top-K over all CUs and the permutation (one
// workgroup up to 512 tokens; histogram, scan and scatter above)
hipError_t launch_route_select(const float *L, const RouteOut &o, int32_t *blockhist, int T, int K, int E,
                               hipStream_t s);
hipError_t init_route_attributes();
hipError_t init_tile_attributes();
// decode routing for 1 <= T <= 16 tokens (bf16) in one launch: logits plus
// bias to L, then, in the last workgroup to finish, top-K, softmax and
// permutation.  `arrive` is a zero device word that the launch leaves zero;
// launches that share it must not overlap.
hipError_t launch_route_decode(const uint16_t *x, const uint16_t *wr, const float *bias, float *L,
                               uint32_t *arrive, const RouteOut &o, int T, int d, int K, int E, hipStream_t s);

// ---- expert projections (experts.hip).  `items` lists the experts of one
// launch (device memory), `n_tiles` the launch's total tile count.
struct ExpertLaunch {
    const WorkItem *items;
    int n_items;
    int n_tiles;
    const void *x;               // [T, d] hidden states (bf16 or f32)
    const void *xh;              // quantized mix, tile path: the hidden states as scaled fp16 and
    const int8_t *xexp;          // their rows' exponents (launch_kq_rows_f16)
    const int32_t *perm;         // gather map of routed rows
    const uint8_t *wbase;        // slot pool
    uint64_t wstride;
    // items with slot < 0 are the shared expert: weights at shared_w, rows
    // are tokens (no gather), act / y go to act_s / ys, weight 1
    const uint8_t *shared_w;
    void *act_s;
    void *ys;                    // [T, d] shared-expert output (bf16; f32 for f32 layers)
    const uint32_t *gen_dev;
    uint32_t *status;
    void *act;                   // [rows, I] bf16 (f32 for f32 layers)
    void *y;                     // [rows, d] weighted expert outputs (bf16; f32 for f32 layers)
    const float *row_weight;     // per permuted row, or null (1.0)
    int d, I;
    // device-built work list (stream kernels only): items resolved by each
    // workgroup from the routing's demanded experts and the residency table;
    // the grid (n_tiles) is then an upper bound and workgroups past the last
    // item exit.  direct.demand null: `items` is the list.
    DirectList direct;
    // device-built work list: when set, the list's length (items, tiles) is
    // read from here and the grid (n_tiles on the host) is an upper bound
    const DevCount *dev_n;
    // router logits launches (ring tiles in router mode) only: x [T, d] tokens,
    // wbase the router weight [E, d], logits[t, e] = x[t] . Wr[e] + bias[e]
    const float *bias;
    float *logits;
    int T, E;
};

// Tile of this workgroup and the launch's work counts: from the device-built
// list (L.dev_n; the grid is an upper bound, tiles spread over the XCDs by
// the real count) or the host list (the grid is the tile count); -1 if this
// workgroup has no tile.  (Scalar loads: the counts are uniform.)
__device__ __forceinline__ int launch_tile(const ExpertLaunch &L, int b, int n_blocks, int &n_items, int &n_tiles)
{
    if (L.dev_n) {
        n_items = __builtin_amdgcn_readfirstlane(L.dev_n->n_items);
        n_tiles = __builtin_amdgcn_readfirstlane(L.dev_n->n_tiles);
        return xcd_tile(b, n_tiles);
    }
    n_items = L.n_items;
    n_tiles = L.n_tiles;
    return xcd_swizzle(b, n_blocks);
}
__device__ __forceinline__ int launch_tile(const ExpertLaunch &L, int &n_items, int &n_tiles)
{
    return launch_tile(L, int(blockIdx.x), int(gridDim.x), n_items, n_tiles);
}

// The tile-path and the stream-path list of a forward in one launch: the first
// tile_blocks workgroups (a multiple of 8, so both lists keep their XCDs) are
// the tile list's.  Few tiles (the shared expert's and those of the busiest
// experts of a small batch) reach few CUs and last as long as a tile does; run
// beside the stream list they cost little, and a launch and its drain go.
// Tile and Stream: run(L, block, blocks, lds), 256 threads, LDS bytes.  Only
// for device-built lists, whose grids bound the tiles instead of counting them.
template <class Tile, class Stream>
__global__ void __launch_bounds__(256, Tile::WAVES_PER_SIMD < Stream::WAVES_PER_SIMD ? Tile::WAVES_PER_SIMD
                                                                                     : Stream::WAVES_PER_SIMD)
    both_kernel(ExpertLaunch T, ExpertLaunch S, int tile_blocks)
{
    extern __shared__ __attribute__((aligned(1024))) uint8_t both_lds[];
    const int b = int(blockIdx.x);
    if (b < tile_blocks)
        Tile::run(T, b, tile_blocks, both_lds);
    else
        Stream::run(S, b - tile_blocks, int(gridDim.x) - tile_blocks, both_lds);
}

template <class Tile, class Stream>
inline hipError_t launch_both(const ExpertLaunch &T, const ExpertLaunch &S, hipStream_t s)
{
    constexpr size_t LDS = Tile::LDS > Stream::LDS ? Tile::LDS : Stream::LDS;
    if (!T.dev_n || !S.dev_n || T.n_tiles % 8 != 0)
        return hipErrorInvalidValue;
    static_assert(LDS <= 64 * 1024, "within the default limit of a launch's LDS");
    launch_k(both_kernel<Tile, Stream>, T.n_tiles + S.n_tiles, 256, LDS, s, T, S, T.n_tiles);
    return hipGetLastError();
}

// Row and weight-slice geometry of a tile-path launch kind: an item of n
// rows has ceil(n / rows) * slices tiles.
struct TileGeom {
    int rows, slices;
};
TileGeom geom_gateup_tile(int d, int I);
TileGeom geom_down_tile(int d, int I);

// Device-built work list of a forward whose demanded experts are all
// published (build_worklist_kernel): the four launch lists (tile and stream
// path, gate/up and down), each ascending by expert, the shared expert first
// in the tile lists, with their counts.
struct WorklistArgs {
    const int32_t *counts, *offsets;     // routing
    const int32_t *slot_of;              // [E] published global slot, -1 if none
    const uint32_t *gen_of;              // [E] published generation
    uint32_t *status;                    // STATUS_MISS if a demanded expert is unpublished
    WorkItem *items[4];                  // gate/up tile, down tile, gate/up stream, down stream; E + 1 each
    DevCount *counts_out;                // [4]
    int E, T, thr, has_shared;
    int clear_status;                    // zero the status word first (the last forward left it set)
    TileGeom gu, dn;                     // tile-path geometry
    int per_gu_stream, per_dn_stream;    // tiles per stream item
};
hipError_t launch_build_worklist(const WorklistArgs &A, hipStream_t s);

// tiles per item of each launch kind
int tiles_gateup_tile(int nrows, int d, int I);
int tiles_down_tile(int nrows, int d, int I);
int tiles_gateup_stream(int nrows, int d, int I);
int tiles_down_stream(int nrows, int d, int I);
int tiles_gateup_f32(int nrows, int d, int I);
int tiles_down_f32(int nrows, int d, int I);

hipError_t launch_gateup_tile(const ExpertLaunch &L, hipStream_t s);
hipError_t launch_down_tile(const ExpertLaunch &L, hipStream_t s);
hipError_t launch_gateup_stream(const ExpertLaunch &L, hipStream_t s);
hipError_t launch_down_stream(const ExpertLaunch &L, hipStream_t s);
hipError_t launch_down_stream_staged(const ExpertLaunch &L, hipStream_t s);
hipError_t launch_gateup_both(const ExpertLaunch &T, const ExpertLaunch &S, hipStream_t s);
hipError_t launch_gateup_f32(const ExpertLaunch &L, hipStream_t s);
hipError_t launch_down_f32(const ExpertLaunch &L, hipStream_t s);

// 4-bit block-quantized experts (experts_q4.hip)
hipError_t init_q4_attributes();

// quantized-expert mix, Wg / Wu in k4 and Wd in k6 (experts_kq.hip)
// xh[t] = fp16(2^xexp[t] x[t]) in the k4 tiles' element order; xexp[t] = KQ_INEXACT: fp16 does not hold the row, and
// the tiles compute it from x
constexpr int8_t KQ_INEXACT = -128;
// (`tiles`: nothing is done if that device-built list is empty; null: always)
hipError_t launch_kq_rows_f16(const void *x, void *xh, int8_t *xexp, int T, int d, const DevCount *tiles, hipStream_t s);
hipError_t init_kq_attributes();

// The expert kernels of one storage format: the tile path (rows above the
// stream threshold, and every row of an f32 layer) and the stream path, for
// gate/up and down, with their tiles per item and tile geometry.  f32 layers
// have no stream path and no device-built lists (null entries).
struct KernelSet {
    using Tiles = int (*)(int nrows, int d, int I);
    using Geom = TileGeom (*)(int d, int I);
    using Launch = hipError_t (*)(const ExpertLaunch &L, hipStream_t s);
    Tiles tiles_gu_tile, tiles_gu_stream, tiles_dn_tile, tiles_dn_stream;
    Geom geom_gu, geom_dn;
    Launch gu_tile, gu_stream, dn_tile, dn_stream;
    // tile and stream list of a device-built pair in one launch, or null
    using Both = hipError_t (*)(const ExpertLaunch &tile, const ExpertLaunch &stream, hipStream_t s);
    Both gu_both = nullptr, dn_both = nullptr;
};
// kernels of a batch of `rows` routed rows (T * K) over E experts, no launch with more than `items` stream items
const KernelSet &q4_kernels(uint64_t rows, uint64_t E, uint64_t items);
const KernelSet &kq_kernels(uint64_t rows, uint64_t E, uint64_t items);
const KernelSet &bf16_kernels(uint64_t rows, uint64_t E);

// ---- combine / publication and slot generation words (combine.hip)
// Status word of a forward and where the combine publishes it.
struct CombinePublish {
    uint32_t *status;            // device status word
    uint32_t *arrive;            // zero device word, left zero: the last workgroup to read the status
                                 // clears it; or null (large grids): the word is left as it is
    uint32_t *host;              // pinned host words (device-visible address), or null:
                                 // [0] status | STATUS_DONE, then, with demand, [1] count, [2..] ids
    const int32_t *demand;       // routing's demanded experts, or null
};
// out[t] = ys[t] + sum_k y[inv[t, k]] in that order (y, ys bf16, or fp32 when
// f32), unless the status word is nonzero
hipError_t launch_combine(const void *y, const void *ys, bool f32, const int32_t *inv, float *out,
                          const CombinePublish &P, int T, int K, int d, hipStream_t s);
constexpr int GEN_BATCH = 64;
struct GenBatch {
    uint32_t n;
    uint32_t slot[GEN_BATCH];
    uint32_t value[GEN_BATCH];
};
hipError_t launch_set_gens(uint32_t *gen_dev, const GenBatch &b, hipStream_t s);
// x0 != null: h = float(x0); else h += out.  Then x = bf16(rmsnorm(h)) per row.
hipError_t launch_residual(const uint16_t *x0, const float *out, float *h, uint16_t *x, int rows, int cols,
                           hipStream_t s);
hipError_t launch_clear_word(uint32_t *word, hipStream_t s);

}  // namespace msi
