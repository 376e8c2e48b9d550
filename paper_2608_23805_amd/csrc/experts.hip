// experts.hip -- per-expert gate/up (SiLU-gated) and down projections for
// gfx950, three variants chosen per expert from its routed-token count only:
//
//  * tile path (bf16, > STREAM tokens): tiles.hip.
//  * stream path (bf16, <= 16 tokens): weight streaming.  The weights are the
//    MFMA A operand, read in whole lines (each wavefront owns 16 weight rows;
//    each weight byte is read once) and rearranged into 16x16x32 fragments in
//    the wavefront's LDS slabs; the expert's tokens (at most 16) are the B
//    operand.
//  * f32 path (fp32 layers): FMA dot products in fixed sequential order
//    (dot_f32.h).
//
// Every workgroup compares the slot generation before its first store and
// writes nothing on a mismatch (fail closed).  Outputs: act[row, I] = silu(x Wg^T) * (x Wu^T) and
// y[row, d] = row_weight * (act Wd^T), rows in permuted order, both rounded
// to bf16 once (fp32 throughout for fp32 layers).
#include "common.h"
#include "dot_f32.h"
#include "gemm_mid.h"
#include "kernels.h"

namespace msi {

// ============================================================== stream path

namespace stream {
constexpr int WAVES = 4;
constexpr int ROWS = 16;        // weight rows per wavefront
}  // namespace stream

int tiles_gateup_stream(int nrows, int d, int I)
{
    (void)nrows;
    (void)d;
    return I / stream::ROWS;
}

int tiles_down_stream(int nrows, int d, int I)
{
    (void)nrows;
    (void)I;
    return d / (stream::WAVES * stream::ROWS);
}

// Stream-path prologue, ordered so that the dependent memory round trips
// before the first MFMA are few: the item is found by division (every stream
// item of a launch has the same tile count), the slot generation word is read
// alongside and checked only before the store (a stale slot is read but
// nothing is written), and the first weight batch is issued before the
// kernel waits for anything else.
struct StreamTile {
    WorkItem it;
    int local;          // tile index within the item
    bool valid;
};

__device__ __forceinline__ StreamTile stream_tile(const ExpertLaunch &L, int per_item, int b, int n_blocks)
{
    StreamTile st{};
    if (L.direct.demand) {
        int i;
        direct_tile(b, per_item, i, st.local);
        if (!direct_item(L.direct, i, per_item, L.status, st.it))
            return st;
        st.valid = st.it.nrows > 0;       // nrows 0: unpublished expert, no work
        return st;
    }
    int n_items, n_tiles;
    const int t = launch_tile(L, b, n_blocks, n_items, n_tiles);
    const int i = t / per_item;
    if (t < 0 || i >= n_items)
        return st;
    st.it = L.items[i];
    st.local = t - i * per_item;
    st.valid = st.it.nrows > 0;
    return st;
}

// Weight slabs.  A wavefront's 16 weight rows reach registers in whole
// 128-byte lines: one 16-byte load per lane covers 8 rows x 128 bytes (lane l:
// row l / 8, chunk l % 8), two loads cover a slab of 16 rows x 64 columns.
// (Loading in the MFMA fragment layout instead, 16 rows x 64 bytes per load,
// reads every line in two halves and streams about 15% slower.)  The slab is
// then rearranged into fragments through the wavefront's own 2 KiB of LDS,
// chunks XOR-swizzled by row so that both the writes and the fragment reads
// are free of bank conflicts.
namespace slab {
constexpr int BYTES = 16 * 128;

// element offset, from the slab's first row and column, of lane's load h (rows 8h .. 8h + 7)
__device__ __forceinline__ int src(int lane, int h, int ld) { return (8 * h + (lane >> 3)) * ld + (lane & 7) * 8; }

// LDS byte offset of the 16 bytes that load h brought to lane
__device__ __forceinline__ int dst(int lane, int h)
{
    const int r = 8 * h + (lane >> 3);
    return r * 128 + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
}

// LDS byte offset of lane's MFMA fragment (row lane % 16, elements 8 (lane / 16) ..) of K step ks (0, 1)
__device__ __forceinline__ int frag(int lane, int ks)
{
    const int r = lane & 15;
    return r * 128 + (((4 * ks + (lane >> 4)) ^ ((r >> 1) & 7)) << 4);
}
}  // namespace slab

__device__ __forceinline__ void lds_wait()
{
    __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0): this wavefront's LDS accesses done
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
}

// Gate/up, stream path: a workgroup owns 16 rows of Wg and of Wu; its four
// wavefronts take the four quarters of d (U K steps of 32, U / 2 slabs per
// matrix, per weight batch) and their fp32 partial sums are added in
// wavefront order before SiLU(g) * u.  The weights (A operand) are streamed
// once, in whole lines (weight slabs above); the lanes of token j (B operand)
// read row j of the item straight from x, which stays in the caches (every
// item reads rows of the same few tokens).  Sixteen-row workgroups keep the
// grid many times larger than the number of resident workgroups, so the last
// partial round of the launch is short.
template <int U, int NB>
struct StreamGateUp {
static constexpr int SL = U / 2;                  // slabs per matrix per batch
static constexpr int REGION = 2 * SL * slab::BYTES;
static constexpr size_t LDS = stream::WAVES * REGION + 3 * 2 * 64 * sizeof(f32x4);
static constexpr int WAVES_PER_SIMD = 3;
static __device__ __forceinline__ void run(const ExpertLaunch &L, int block, int n_blocks, uint8_t *lds)
{
    f32x4 (*red)[2][64] = reinterpret_cast<f32x4 (*)[2][64]>(lds + stream::WAVES * REGION);
    const int d = L.d, I = L.I;
    const StreamTile st = stream_tile(L, I / stream::ROWS, block, n_blocks);
    if (!st.valid)
        return;
    const WorkItem &it = st.it;
    const int n = it.nrows;
    const bool sh = it.slot < 0;
    const uint32_t gnow = slot_gen_now(it, L.gen_dev);

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int i0 = st.local * stream::ROWS;
    const int kq = d / stream::WAVES;             // this wavefront's quarter of d
    const int j = lane & 15, kg = (lane >> 4) * 8;
    const uint8_t *base = sh ? L.shared_w : L.wbase + uint64_t(it.slot) * L.wstride;
    const uint16_t *w0 = reinterpret_cast<const uint16_t *>(base) + int64_t(i0) * d + wave * kq;
    const uint16_t *gp0 = w0 + slab::src(lane, 0, d), *gp1 = w0 + slab::src(lane, 1, d);
    const int64_t um = int64_t(I) * d;            // Wu follows Wg
    const bool live = j < n;
    uint8_t *t = lds + wave * REGION;

    // This lane's token (the shared expert's rows are the tokens in order),
    // read before the weights are issued: memory reads complete in order, so
    // waiting for it later leaves the weight batch in flight.  Lanes past
    // the item's rows read its last row: an MFMA output column depends only
    // on its own B column, and those columns are never stored.  Every read is
    // unconditional, so the compiler's waits stay exact.
    const int jr = it.row0 + min(j, n - 1);
    const int64_t xrow = sh ? int64_t(jr) : int64_t(L.perm[jr]);
    // The quarter goes in chunks of NB batches, each fully unrolled: weight
    // and token batches are double-buffered in registers (batch b + 1 is in
    // flight while batch b is rearranged and multiplied), and with no
    // register live across chunks the compiler's memory waits stay exact.
    // (The empty asm statements keep the issue order: token index, weights,
    // token rows.)
    const uint16_t *xp = reinterpret_cast<const uint16_t *>(L.x) + xrow * d + wave * kq + kg;
    auto load_w = [&](u32x4(&dst)[2][SL][2], int k0) {
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int s = 0; s < SL; ++s) {
                dst[m][s][0] = load_stream16(gp0 + m * um + k0 + 64 * s);
                dst[m][s][1] = load_stream16(gp1 + m * um + k0 + 64 * s);
            }
    };
    auto load_x = [&](u32x4(&dst)[U], int k0) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            dst[u] = *reinterpret_cast<const u32x4 *>(xp + k0 + 32 * u);
    };
    f32x4 ag = {0.f, 0.f, 0.f, 0.f}, au = {0.f, 0.f, 0.f, 0.f};
    const int nchunk = kq / (32 * U * NB);
    for (int c = 0; c < nchunk; ++c) {
        const int kc = c * 32 * U * NB;
        u32x4 w[2][2][SL][2], xb[2][U];               // [buffer][matrix][slab][load]
        asm volatile("" ::: "memory");
        load_w(w[0], kc);
        asm volatile("" ::: "memory");
        load_x(xb[0], kc);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (b + 1 < NB) {
                load_w(w[(b + 1) & 1], kc + (b + 1) * 32 * U);
                load_x(xb[(b + 1) & 1], kc + (b + 1) * 32 * U);
            }
            // rearrange batch b into fragments
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int s = 0; s < SL; ++s)
#pragma unroll
                    for (int q = 0; q < 2; ++q)
                        *reinterpret_cast<u32x4 *>(t + (m * SL + s) * slab::BYTES + slab::dst(lane, q)) =
                            w[b & 1][m][s][q];
            lds_wait();
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bf16x8 bx = as_bf16x8(xb[b & 1][u]);
                const u32x4 fg =
                    *reinterpret_cast<const u32x4 *>(t + (u >> 1) * slab::BYTES + slab::frag(lane, u & 1));
                const u32x4 fu =
                    *reinterpret_cast<const u32x4 *>(t + (SL + (u >> 1)) * slab::BYTES + slab::frag(lane, u & 1));
                ag = mfma16(as_bf16x8(fg), bx, ag);
                au = mfma16(as_bf16x8(fu), bx, au);
            }
            lds_wait();                               // the next batch overwrites this wavefront's slabs
        }
    }
    // quarters of d added in wavefront order
    if (wave > 0) {
        red[wave - 1][0][lane] = ag;
        red[wave - 1][1][lane] = au;
    }
    __syncthreads();
    if (wave != 0)
        return;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        ag[r] = ((ag[r] + red[0][0][lane][r]) + red[1][0][lane][r]) + red[2][0][lane][r];
        au[r] = ((au[r] + red[0][1][lane][r]) + red[1][1][lane][r]) + red[2][1][lane][r];
    }
    if (!slot_gen_ok(it, gnow, L.status))
        return;
    // lane holds rows i0 + 4*(lane/16) + r of token j
    if (live) {
        uint2 v;
        v.x = pack_bf16x2(silu(ag[0]) * au[0], silu(ag[1]) * au[1]);
        v.y = pack_bf16x2(silu(ag[2]) * au[2], silu(ag[3]) * au[3]);
        uint16_t *act = reinterpret_cast<uint16_t *>(sh ? L.act_s : L.act) + int64_t(it.row0 + j) * I + i0 +
                        4 * (lane >> 4);
        *reinterpret_cast<uint2 *>(act) = v;
    }
}
};

template <int U, int NB>
__global__ void __launch_bounds__(256, 3) stream_gateup_kernel(ExpertLaunch L)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[StreamGateUp<U, NB>::LDS];
    StreamGateUp<U, NB>::run(L, int(blockIdx.x), int(gridDim.x), lds);
}

// Down, stream path: a workgroup owns 64 output columns (16 per wavefront)
// over all of I, in chunks of NB batches of 4 K steps (2 slabs of Wd rows,
// loaded in whole lines and rearranged through the wavefront's LDS as in the
// gate/up kernel), each chunk fully unrolled.  The lanes of token j (B
// operand) read row j of the item's act rows straight from memory with each
// weight batch (the rows are contiguous and few; lanes past the item's rows
// read its last row, whose outputs are never stored), so no workgroup
// barrier or LDS staging comes before the first MFMA.  STAGE: the workgroup
// stages the item's rows in LDS once instead.  The four wavefronts read the
// same rows, and a direct load of 16 of them touches 16 lines for the 8 of a
// weight load; with ten rows and more that costs more than the barrier.
// Measured (MI355X, E 512, d 2048, I 512, K 10; direct / staged, us): 2.5 mean
// rows 141 / 144, 5 161 / 162, 6 167 / 166, 8 178 / 169, 10 186 / 170, 16
// (half of the experts) 129 / 113; I 768, E 128: 8 rows 34 / 35, 12 35 / 33.
namespace stream_down {
constexpr int U = 4, SL = U / 2;
constexpr int REGION = SL * slab::BYTES;
constexpr int LDS = stream::WAVES * REGION;       // the wavefronts' weight slabs
}  // namespace stream_down

template <int NB, bool STAGE>
__global__ void __launch_bounds__(256, 4) stream_down_kernel(ExpertLaunch L)
{
    using namespace stream_down;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int d = L.d, I = L.I;
    const StreamTile st = stream_tile(L, d / (stream::WAVES * stream::ROWS), int(blockIdx.x), int(gridDim.x));
    if (!st.valid)
        return;
    const WorkItem &it = st.it;
    const int n = it.nrows;
    const bool sh = it.slot < 0;
    const uint32_t gnow = slot_gen_now(it, L.gen_dev);

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int c0 = (st.local * stream::WAVES + wave) * stream::ROWS;
    const int j = lane & 15, kg = (lane >> 4) * 8;
    const uint8_t *base = sh ? L.shared_w : L.wbase + uint64_t(it.slot) * L.wstride;
    const uint16_t *w0 = reinterpret_cast<const uint16_t *>(base) + int64_t(2) * I * d + int64_t(c0) * I;
    const uint16_t *gp0 = w0 + slab::src(lane, 0, I), *gp1 = w0 + slab::src(lane, 1, I);
    const uint16_t *ap = reinterpret_cast<const uint16_t *>(sh ? L.act_s : L.act) +
                         int64_t(it.row0 + min(j, n - 1)) * I + kg;
    const bool live = j < n;
    uint8_t *t = lds + wave * REGION;
    auto load_w = [&](u32x4(&dst)[SL][2], u32x4(&adst)[U], int k0) {
#pragma unroll
        for (int s = 0; s < SL; ++s) {
            dst[s][0] = load_stream16(gp0 + k0 + 64 * s);
            dst[s][1] = load_stream16(gp1 + k0 + 64 * s);
        }
        if constexpr (!STAGE)
#pragma unroll
            for (int u = 0; u < U; ++u)
                adst[u] = *reinterpret_cast<const u32x4 *>(ap + k0 + 32 * u);
    };
    u32x4 w[2][SL][2], av[2][U];
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    // staged rows: thread t brings 16-byte piece t % 16 of every 128 columns of row t / 16; the row stride
    // sends the 16 rows' pieces of a fragment read to different banks
    const int sr = 2 * I + 16;
    uint8_t *srow = lds + stream::WAVES * REGION + (threadIdx.x >> 4) * sr + 16 * (threadIdx.x & 15);
    const uint8_t *sfrag = lds + stream::WAVES * REGION + j * sr + 2 * kg;
    const uint16_t *grow = reinterpret_cast<const uint16_t *>(sh ? L.act_s : L.act) +
                           int64_t(it.row0 + min(int(threadIdx.x >> 4), n - 1)) * I + 8 * (threadIdx.x & 15);
    constexpr int NS = 4;                             // pieces loaded ahead of the first weights: 512 columns
    u32x4 sv[NS];
    if constexpr (STAGE)
#pragma unroll
        for (int i = 0; i < NS; ++i)
            if (128 * i < I)
                sv[i] = *reinterpret_cast<const u32x4 *>(grow + 128 * i);
    const int nchunk = I / (32 * U * NB);
    for (int c = 0; c < nchunk; ++c) {
        const int kc = c * 32 * U * NB;
        asm volatile("" ::: "memory");
        load_w(w[0], av[0], kc);
        if (NB > 1)
            load_w(w[1], av[1], kc + 32 * U);
        if (STAGE && c == 0) {
#pragma unroll
            for (int i = 0; i < NS; ++i)
                if (128 * i < I)
                    *reinterpret_cast<u32x4 *>(srow + 256 * i) = sv[i];
            for (int i = NS; 128 * i < I; ++i)
                *reinterpret_cast<u32x4 *>(srow + 256 * i) = *reinterpret_cast<const u32x4 *>(grow + 128 * i);
            __syncthreads();
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (b >= 1 && b + 1 < NB)                 // batches 0 and 1 went out with the chunk
                load_w(w[(b + 1) & 1], av[(b + 1) & 1], kc + (b + 1) * 32 * U);
#pragma unroll
            for (int s = 0; s < SL; ++s)
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    *reinterpret_cast<u32x4 *>(t + s * slab::BYTES + slab::dst(lane, q)) = w[b & 1][s][q];
            lds_wait();
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const u32x4 fw = *reinterpret_cast<const u32x4 *>(t + (u >> 1) * slab::BYTES + slab::frag(lane, u & 1));
                const u32x4 fa = STAGE ? *reinterpret_cast<const u32x4 *>(sfrag + 2 * (kc + 32 * (b * U + u)))
                                       : av[b & 1][u];
                acc = mfma16(as_bf16x8(fw), as_bf16x8(fa), acc);
            }
            lds_wait();                               // the next batch overwrites this wavefront's slabs
        }
    }
    if (!slot_gen_ok(it, gnow, L.status))
        return;
    if (live) {
        const int64_t row = it.row0 + j;
        const float wt = sh ? 1.0f : L.row_weight[row];
        *reinterpret_cast<uint2 *>(static_cast<uint16_t *>(sh ? L.ys : L.y) + row * d + c0 + 4 * (lane >> 4)) =
            make_uint2(pack_bf16x2(acc[0] * wt, acc[1] * wt), pack_bf16x2(acc[2] * wt, acc[3] * wt));
    }
}

hipError_t launch_gateup_stream(const ExpertLaunch &L, hipStream_t s)
{
    if (L.n_tiles == 0)
        return hipSuccess;
    // chunks of NB batches of U K steps of 32 must divide the quarter d / 4 (d % 256 == 0)
    const int kq = L.d / 4;
    if (kq % 512 == 0)
        launch_k(stream_gateup_kernel<4, 4>, L.n_tiles, 256, 0, s, L);
    else if (kq % 256 == 0)
        launch_k(stream_gateup_kernel<4, 2>, L.n_tiles, 256, 0, s, L);
    else if (kq % 128 == 0)
        launch_k(stream_gateup_kernel<4, 1>, L.n_tiles, 256, 0, s, L);
    else
        launch_k(stream_gateup_kernel<2, 1>, L.n_tiles, 256, 0, s, L);
    return hipGetLastError();
}

template <bool STAGE>
static hipError_t launch_down(const ExpertLaunch &L, hipStream_t s)
{
    const int lds = stream_down::LDS + (STAGE ? 16 * (2 * L.I + 16) : 0);
    // chunks of NB batches of 128 columns must divide I (I % 128 == 0)
    if (L.I % 512 == 0)
        launch_k(stream_down_kernel<4, STAGE>, L.n_tiles, 256, lds, s, L);
    else if (L.I % 256 == 0)
        launch_k(stream_down_kernel<2, STAGE>, L.n_tiles, 256, lds, s, L);
    else
        launch_k(stream_down_kernel<1, STAGE>, L.n_tiles, 256, lds, s, L);
    return hipGetLastError();
}

hipError_t launch_down_stream(const ExpertLaunch &L, hipStream_t s)
{
    return L.n_tiles == 0 ? hipSuccess : launch_down<false>(L, s);
}

// Staged where it measured faster at every batch past the rule's 8 mean rows: 16 KB of weight slabs and 32 I + 256
// bytes of rows leave a CU its four workgroups up to I = 640 and three above.  Direct / staged, us (d 2048, K 8, E 256,
// mean rows 9, 10, 12, 14, 16): I 640 115 / 111, 118 / 111, 114 / 107, 100 / 92, 69 / 64; I 768 134 / 130, 137 / 130,
// 136 / 126, 119 / 107, 81 / 74; I 896 156 / 156, 158 / 157, 156 / 150, 136 / 129, 92 / 90, but at E 128 78 / 81,
// 79 / 81, 76 / 74, 66 / 67, 50 / 47 (I 768 there 68 / 67, 68 / 67, 66 / 62, 58 / 54, 43 / 39).
hipError_t launch_down_stream_staged(const ExpertLaunch &L, hipStream_t s)
{
    return L.n_tiles == 0 ? hipSuccess : L.I <= 768 ? launch_down<true>(L, s) : launch_down<false>(L, s);
}

// The 64-row tiles and the stream list in one launch (both_kernel).  Measured
// (MI355X, E 512, d 2048, I 512, K 10; gate/up, us): two launches 15.7 + 276
// (128 tokens), 17.6 + 302 (509), 146 + 200 (800); together 282, 313, 340.
// The tiles keep two stage buffers here, not three: 49 KB of LDS, so that
// three workgroups of either list share a CU (the stream list's own three).
// Down stays in two launches: its stream kernel runs four workgroups per CU
// and lost more at three (203 against 9.6 + 186 us at 509 tokens).
hipError_t launch_gateup_both(const ExpertLaunch &T, const ExpertLaunch &S, hipStream_t s)
{
    using Tile = MidTile<RingMode::GateUp, Mid64Both>;
    const int kq = S.d / 4;
    if (kq % 512 == 0)
        return launch_both<Tile, StreamGateUp<4, 4>>(T, S, s);
    if (kq % 256 == 0)
        return launch_both<Tile, StreamGateUp<4, 2>>(T, S, s);
    if (kq % 128 == 0)
        return launch_both<Tile, StreamGateUp<4, 1>>(T, S, s);
    return launch_both<Tile, StreamGateUp<2, 1>>(T, S, s);
}

// ============================================================== f32 path

int tiles_gateup_f32(int nrows, int d, int I)
{
    (void)d;
    return ((nrows + f32t::ROWS - 1) / f32t::ROWS) * (I / f32t::COLS);
}

int tiles_down_f32(int nrows, int d, int I)
{
    (void)I;
    return ((nrows + f32t::ROWS - 1) / f32t::ROWS) * (d / f32t::COLS);
}

__global__ void __launch_bounds__(256) gateup_f32_kernel(ExpertLaunch L)
{
    __shared__ f32t::Stage<2> lds;
    const int t = xcd_swizzle(int(blockIdx.x), int(gridDim.x));
    const WorkItem it = L.items[find_item(L.items, L.n_items, t)];
    if (!slot_current(it, L.gen_dev, L.status))
        return;
    const int d = L.d, I = L.I;
    const int local = t - it.tile0, nct = I / f32t::COLS;
    const int m0 = (local / nct) * f32t::ROWS, c0 = (local % nct) * f32t::COLS;
    const bool sh = it.slot < 0;
    const uint8_t *base = sh ? L.shared_w : L.wbase + uint64_t(it.slot) * L.wstride;
    const float *w[2];
    w[0] = reinterpret_cast<const float *>(base) + int64_t(c0) * d;
    w[1] = w[0] + int64_t(I) * d;
    float acc[2];
    f32t::dot<2>(lds, [&](int q) {
        const int r = it.row0 + min(m0 + q, it.nrows - 1);
        return reinterpret_cast<const float *>(L.x) + (sh ? int64_t(r) : int64_t(L.perm[r])) * d;
    }, w, [](int c) { return c; }, d, acc);
    const int r = m0 + int(threadIdx.x) / f32t::COLS, c = c0 + int(threadIdx.x) % f32t::COLS;
    if (r < it.nrows)
        reinterpret_cast<float *>(sh ? L.act_s : L.act)[int64_t(it.row0 + r) * I + c] = silu(acc[0]) * acc[1];
}

__global__ void __launch_bounds__(256) down_f32_kernel(ExpertLaunch L)
{
    __shared__ f32t::Stage<1> lds;
    const int t = xcd_swizzle(int(blockIdx.x), int(gridDim.x));
    const WorkItem it = L.items[find_item(L.items, L.n_items, t)];
    if (!slot_current(it, L.gen_dev, L.status))
        return;
    const int d = L.d, I = L.I;
    const int local = t - it.tile0, nct = d / f32t::COLS;
    const int m0 = (local / nct) * f32t::ROWS, c0 = (local % nct) * f32t::COLS;
    const bool sh = it.slot < 0;
    const uint8_t *base = sh ? L.shared_w : L.wbase + uint64_t(it.slot) * L.wstride;
    const float *w[1] = {reinterpret_cast<const float *>(base) + int64_t(2) * I * d + int64_t(c0) * I};
    float acc[1];
    f32t::dot<1>(lds, [&](int q) {
        return reinterpret_cast<const float *>(sh ? L.act_s : L.act) +
               int64_t(it.row0 + min(m0 + q, it.nrows - 1)) * I;
    }, w, [](int c) { return c; }, I, acc);
    const int r = m0 + int(threadIdx.x) / f32t::COLS, c = c0 + int(threadIdx.x) % f32t::COLS;
    if (r < it.nrows) {
        const int64_t row = it.row0 + r;
        const float wt = sh ? 1.0f : L.row_weight[row];
        static_cast<float *>(sh ? L.ys : L.y)[row * d + c] = acc[0] * wt;
    }
}

hipError_t launch_gateup_f32(const ExpertLaunch &L, hipStream_t s)
{
    if (L.n_tiles == 0)
        return hipSuccess;
    launch_k(gateup_f32_kernel, L.n_tiles, 256, 0, s, L);
    return hipGetLastError();
}

hipError_t launch_down_f32(const ExpertLaunch &L, hipStream_t s)
{
    if (L.n_tiles == 0)
        return hipSuccess;
    launch_k(down_f32_kernel, L.n_tiles, 256, 0, s, L);
    return hipGetLastError();
}

}  // namespace msi

namespace msi {

hipError_t init_kernel_attributes()
{
    hipError_t e = init_tile_attributes();
    if (e == hipSuccess)
        e = init_route_attributes();
    if (e == hipSuccess)
        e = init_q4_attributes();
    if (e == hipSuccess)
        e = init_kq_attributes();
    return e;
}

}  // namespace msi
