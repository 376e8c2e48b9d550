// tiles.hip -- launches of the tile kernels (gemm_ring.h, gemm_mid.h): the
// routed-expert gate/up and down projections of experts with more than 16
// routed rows, and the router logits of batches of more than 16 tokens.
#include "common.h"
#include "gemm_mid.h"
#include "gemm_ring.h"
#include "kernels.h"

namespace msi {

int tiles_gateup_tile(int nrows, int d, int I)
{
    (void)d;
    return ring_tiles_gateup(nrows, I);
}

int tiles_down_tile(int nrows, int d, int I)
{
    (void)I;
    return ring_tiles_down(nrows, d);
}

TileGeom geom_gateup_tile(int d, int I)
{
    (void)d;
    return TileGeom{ring::TM, I / 128};
}

TileGeom geom_down_tile(int d, int I)
{
    (void)I;
    return TileGeom{ring::TM, d / ring::TN};
}

// Shapes of the tile path for few rows per expert (bf16_kernels holds the rule between them and the 256-row
// form), and of the router logits.
using Mid128 = MidShape<128, 256, 2, 4, 3, 1>;
using Router32 = MidShape<32, 32, 2, 2, 6, 1>;
using Router64 = MidShape<64, 64, 2, 2, 4, 2>;

template <class S>
static int tiles_gateup_mid(int nrows, int, int I)
{
    return (nrows + S::BM - 1) / S::BM * (I / (S::TN / 2));
}

template <class S>
static int tiles_down_mid(int nrows, int d, int)
{
    return (nrows + S::BM - 1) / S::BM * (d / S::TN);
}

template <class S>
static TileGeom geom_gateup_mid(int, int I)
{
    return TileGeom{S::BM, I / (S::TN / 2)};
}

template <class S>
static TileGeom geom_down_mid(int d, int)
{
    return TileGeom{S::BM, d / S::TN};
}

template <RingMode M, class S>
static hipError_t launch_mid(const ExpertLaunch &L, hipStream_t s)
{
    if (L.n_tiles == 0)
        return hipSuccess;
    launch_k(mid_gemm_kernel<M, S>, L.n_tiles, S::THREADS, S::LDS, s, L);
    return hipGetLastError();
}

template <class S, bool STAGE>
static const KernelSet mid_set{tiles_gateup_mid<S>, tiles_gateup_stream, tiles_down_mid<S>, tiles_down_stream,
                               geom_gateup_mid<S>, geom_down_mid<S>,
                               launch_mid<RingMode::GateUp, S>, launch_gateup_stream,
                               launch_mid<RingMode::Down, S>,
                               STAGE ? launch_down_stream_staged : launch_down_stream,
                               S::BM == Mid64Both::BM ? launch_gateup_both : nullptr};

// The tile path's form by the mean rows per expert.  The three are
// bit-identical, so the choice is the launch's and no result depends on it.
// Measured (MI355X, E 512, d 2048, I 512, K 10; gate/up + down, us):
//   mean rows   64-row   128-row   256-row
//      20       278+165  302+172   311+191
//      40       390+232  400+235   430+256
//      80       523+290  411+261   469+280
//     160       692+420  591+382   533+348
// (below 64 rows the 64-row form streams the weights with two workgroups per
// CU; past it most experts need two of its tiles, each reading the weights.)
// Past 8 mean rows the stream list's down stages its act rows (both sides are
// at its kernel).
const KernelSet &bf16_kernels(uint64_t rows, uint64_t E)
{
    static const KernelSet ring256{tiles_gateup_tile, tiles_gateup_stream, tiles_down_tile, tiles_down_stream,
                                   geom_gateup_tile, geom_down_tile,
                                   launch_gateup_tile, launch_gateup_stream, launch_down_tile, launch_down_stream_staged};
    if (rows <= 48 * E)
        return rows <= 8 * E ? mid_set<Mid64, false> : mid_set<Mid64, true>;
    return rows <= 112 * E ? mid_set<Mid128, true> : ring256;
}

// workgroups of a persistent launch: one per compute unit
static int g_persistent_wgs = 256;

hipError_t launch_gateup_tile(const ExpertLaunch &L, hipStream_t s)
{
    if (L.n_tiles == 0)
        return hipSuccess;
    // (the persistent form is slower for gate/up: its extra state spills registers, and the spill reloads
    // wait for every copy in flight)
    launch_k(ring_gemm_kernel<RingMode::GateUp>, L.n_tiles, ring::THREADS, 0, s, L);
    return hipGetLastError();
}

hipError_t launch_down_tile(const ExpertLaunch &L, hipStream_t s)
{
    if (L.n_tiles == 0)
        return hipSuccess;
    if ((L.I / ring::SK) % 4 == 0 && L.I / ring::SK >= 8 && L.n_tiles > g_persistent_wgs) {
        // K loop long enough for the cross-tile pipeline: one workgroup per CU walks its tiles
        launch_k(ring_gemm_persistent<RingMode::Down>, g_persistent_wgs, ring::THREADS, 0, s, L);
    } else {
        launch_k(ring_gemm_kernel<RingMode::Down>, L.n_tiles, ring::THREADS, 0, s, L);
    }
    return hipGetLastError();
}

hipError_t launch_router_logits_bf16(const uint16_t *x, const uint16_t *wr, const float *bias, float *L, int T,
                                     int d, int E, hipStream_t s)
{
    if (T == 0)
        return hipSuccess;
    ExpertLaunch R{};
    R.x = x;
    R.wbase = reinterpret_cast<const uint8_t *>(wr);
    R.d = d;
    R.bias = bias;
    R.logits = L;
    R.T = T;
    R.E = E;
    // A workgroup copies its rows to LDS at about 50 bytes/ns, so a tile costs what its rows do (64 + 128 rows of
    // 4 KiB: 16 us) however few tiles there are.  The smallest tiles that fit in two per CU are taken, and the
    // 256 x 256 form above that; all are bit-identical.  Measured (E 512, d 2048, us: 32 x 32, 64 x 64,
    // 64 x 128, 256 x 256): T 251 8.3, 12.9, 19.3, 47; T 1024 12.4, 15.0, 21.6, 58; T 4096 34.0, 21.8, 21.8,
    // 58; T 8192 63.6, 41.7, 34.5, 59; T 16384 -, -, 85, 63.
    auto tiles_of = [&](int bm, int tn) { return ((T + bm - 1) / bm) * ((E + tn - 1) / tn); };
    constexpr int MAX_TILES = 512;
    auto mid = [&](auto shape) {
        using S = decltype(shape);
        R.n_tiles = tiles_of(S::BM, S::TN);
        return launch_mid<RingMode::Router, S>(R, s);
    };
    if (tiles_of(32, 32) <= MAX_TILES)
        return mid(Router32{});
    if (tiles_of(64, 64) <= MAX_TILES)
        return mid(Router64{});
    if (tiles_of(64, 128) <= MAX_TILES)
        return mid(Mid64{});
    launch_k(ring_gemm_kernel<RingMode::Router>, tiles_of(ring::TM, ring::TN), ring::THREADS, 0, s, R);
    return hipGetLastError();
}

hipError_t init_tile_attributes()
{
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess)
        e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess)
        return e;
    for (const void *f : {reinterpret_cast<const void *>(&mid_gemm_kernel<RingMode::GateUp, Mid64>),
                          reinterpret_cast<const void *>(&mid_gemm_kernel<RingMode::Down, Mid64>),
                          reinterpret_cast<const void *>(&mid_gemm_kernel<RingMode::GateUp, Mid128>),
                          reinterpret_cast<const void *>(&mid_gemm_kernel<RingMode::Down, Mid128>),
                          reinterpret_cast<const void *>(&mid_gemm_kernel<RingMode::Router, Mid64>),
                          reinterpret_cast<const void *>(&mid_gemm_kernel<RingMode::Router, Router32>),
                          reinterpret_cast<const void *>(&mid_gemm_kernel<RingMode::Router, Router64>)})
        if ((e = allow_large_lds(f)) != hipSuccess)
            return e;
    // a multiple of the 8 XCDs keeps each XCD's workgroups on its own tile range
    g_persistent_wgs = cus >= 8 ? cus / 8 * 8 : 8;
    return hipSuccess;
}

}  // namespace msi
