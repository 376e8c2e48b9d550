// experts_q4.hip -- 4-bit block-quantized expert projections for gfx950.
//
// Storage (per matrix [rows, cols]): nibbles [rows, cols/2] (element 2j in the
// low nibble of byte j, 4-bit two's complement) then fp16 scales
// [rows, cols/32]; value = scale * q.  Every 16x16x32 MFMA spans exactly one
// 32-element scale block, so it returns the block's partial dot product and
// the scale is applied in fp32: acc += scale * partial.
//
//  * stream path (<= 16 tokens per expert): tokens as the A operand and
//    weights as the B operand, tokens read straight from memory and the
//    nibbles through row-contiguous loads rearranged in LDS (WaveRows); the
//    codes unpacked to exact bf16 q / 16 (C = 0).
//  * tile path: 64 or 128 tokens x 128 weight rows per workgroup; token rows,
//    packed nibbles and scales copied from memory straight into two LDS stage
//    buffers; the codes enter the MFMA as the exact bf16 136 + q, and the
//    offset leaves through the C input (-136 times the token row's block sum,
//    from one more MFMA per token fragment).
#include "common.h"
#include "gemm_ring.h"
#include "kernels.h"

namespace msi {

__device__ __forceinline__ uint32_t q4_matrix_bytes(int rows, int cols)
{
    return uint32_t(rows) * uint32_t(cols / 2) + uint32_t(rows) * uint32_t(cols / 32) * 2u;
}

// 8 nibbles (element e at bits 4e..4e+3, two's complement q) -> 8 exact bf16
// values 136 + q: the bits 0x4300 | u are the bf16 128 + u, u = q + 8 = the
// nibble with its top bit flipped.  Byte permutes place the nibbles (even
// elements from the low halves of the bytes, odd ones from the high halves)
// under the 0x43 bytes: nine operations per 8 values.
__device__ __forceinline__ bf16x8 unpack_q4_136(uint32_t w)
{
    const uint32_t e = (w ^ 0x08080808u) & 0x0F0F0F0Fu;           // u of elements 0, 2, 4, 6
    const uint32_t o = ((w >> 4) ^ 0x08080808u) & 0x0F0F0F0Fu;    // u of elements 1, 3, 5, 7
    const uint32_t lo = __builtin_amdgcn_perm(o, e, 0x05010400u);  // bytes u0 u1 u2 u3
    const uint32_t hi = __builtin_amdgcn_perm(o, e, 0x07030602u);  // bytes u4 u5 u6 u7
    u32x4 r;
    r[0] = __builtin_amdgcn_perm(0x43434343u, lo, 0x04010400u);
    r[1] = __builtin_amdgcn_perm(0x43434343u, lo, 0x04030402u);
    r[2] = __builtin_amdgcn_perm(0x43434343u, hi, 0x04010400u);
    r[3] = __builtin_amdgcn_perm(0x43434343u, hi, 0x04030402u);
    return __builtin_bit_cast(bf16x8, r);
}

// 8 nibbles (element e at bits 4e..4e+3, two's complement q) -> 8 exact bf16
// values q / 16: the 4-bit integer conversion reads the low nibble of a byte
// and returns q / 16 in binary32, whose top half holds it; thirteen operations
// per 8 values.
__device__ __forceinline__ bf16x8 unpack_q4_16th(uint32_t w)
{
    uint32_t o = w >> 4;
    asm("" : "+v"(o));          // (one shift; the conversions then pick their byte of it)
    u32x4 r;
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const float fe = __builtin_amdgcn_cvt_off_f32_i4(int((w >> (8 * h)) & 0xFFu));   // element 2h
        const float fo = __builtin_amdgcn_cvt_off_f32_i4(int((o >> (8 * h)) & 0xFFu));   // element 2h + 1
        r[h] = __builtin_amdgcn_perm(__float_as_uint(fo), __float_as_uint(fe), 0x07060302u);
    }
    return __builtin_bit_cast(bf16x8, r);
}

__device__ __forceinline__ float half_to_float(uint16_t h) { return float(__builtin_bit_cast(_Float16, h)); }

// ============================================================== stream path

namespace q4s {
constexpr int WAVES = 4, ROWS = 16;
}

// Tile t of a stream launch and its item: from the device-built list (the
// grid is then an upper bound) or the host list.
__device__ __forceinline__ bool q4_tile(const ExpertLaunch &L, int per_item, int b, int n_blocks, int &t, WorkItem &it)
{
    if (L.direct.demand) {
        int i, local;
        direct_tile(b, per_item, i, local);
        t = i * per_item + local;
        return direct_item(L.direct, i, per_item, L.status, it);
    }
    int n_items, n_tiles;
    t = launch_tile(L, b, n_blocks, n_items, n_tiles);
    if (t < 0)
        return false;
    it = L.items[find_item(L.items, n_items, t)];
    return true;
}

// CH consecutive fp16 block scales of one row, in one vector load (the
// row's scales start 16-byte aligned and CH divides the blocks of a quarter
// of d, or of I).
template <int CH>
__device__ __forceinline__ void load_scales(uint32_t (&w)[CH / 2], const uint16_t *p)
{
    if constexpr (CH == 8) {
        const u32x4 a = *reinterpret_cast<const u32x4 *>(p);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            w[i] = a[i];
    } else if constexpr (CH == 4) {
        const uint2 a = *reinterpret_cast<const uint2 *>(p);
        w[0] = a.x;
        w[1] = a.y;
    } else {
        w[0] = *reinterpret_cast<const uint32_t *>(p);
    }
}

__device__ __forceinline__ float scale_at(const uint32_t *w, int b)
{
    return half_to_float(uint16_t(w[b >> 1] >> (16 * (b & 1))));
}

// Gate/up, 4-bit stream path: a workgroup owns 16 R rows of Wg and of Wu; its
// four wavefronts take the four quarters of d and add their fp32 partial sums
// in wavefront order before SiLU(g) * u, so an item is I / (16 R) workgroups.
// Tokens are the A operand and weights the B operand: lane (r = lane % 16,
// g = lane / 16) holds elements 8g .. 8g + 7 of each block of token r and of
// weight rows i0 + 16 q + r, and its outputs are tokens 4g .. 4g + 3 of those
// rows, so each lane applies its rows' block scales.  Token fragments come
// straight from global memory (lanes past the item's rows repeat its last
// row and are not stored); the nibbles go through WaveRows (row-contiguous
// 16-byte loads, rearranged in the wavefront's own LDS region).  Blocks go
// in chunks of CH, each chunk's loads issued before its first MFMA.  The sums
// are sixteenths (exact: a power of two) until they are whole.  A token
// fragment is 1 KiB from 16 rows, which R = 1 gives to 512 bytes of codes and
// R = 2 to 1 KiB; alone the two forms stay within 2 us of each other, beside
// the tile list R = 2 gains 9% (both at q4_kernels).
template <int CH, int R>
struct Q4StreamGateUp {
using Rows = WaveRows<16 * CH>;
static constexpr int NM = 2 * R;                       // 16-row groups: R of Wg, then R of Wu
static constexpr int REGION = NM * 16 * Rows::RS > NM * 1024 ? NM * 16 * Rows::RS : NM * 1024;
static constexpr size_t LDS = q4s::WAVES * REGION;
static constexpr int WAVES_PER_SIMD = 3;
static __device__ __forceinline__ void run(const ExpertLaunch &L, int block, int n_blocks, uint8_t *lds)
{
    // a wavefront's rows, then (its own part) its partial sums
    uint8_t (*wst)[REGION] = reinterpret_cast<uint8_t (*)[REGION]>(lds);
    const int d = L.d, I = L.I, nblk = d / 32, nq = nblk / q4s::WAVES;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, g = lane >> 4;
    const int bq = wave * nq;                          // this wavefront's first block
    // One token (a device-built decode list of T = 1): every row is token 0, so the token fragments of the
    // first chunk are requested before the item is known, and the generation is compared after the work
    // (before the stores), so the weights are requested as soon as the slot is known.
    const bool one = L.direct.demand && L.direct.T == 1;
    u32x4 xv[CH];
    if (one) {
#pragma unroll
        for (int u = 0; u < CH; ++u)
            xv[u] = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const uint16_t *>(L.x) + 8 * g + 32 * (bq + u));
    }
    int t;
    WorkItem it;
    if (!q4_tile(L, I / (q4s::ROWS * R), block, n_blocks, t, it) || it.nrows == 0)   // nrows 0: unpublished expert, no work
        return;
    const uint32_t gnow = slot_gen_now(it, L.gen_dev);
    const int n = it.nrows;
    const bool sh = it.slot < 0;
    const int i0 = (t - it.tile0) * q4s::ROWS * R;
    const uint8_t *base = sh ? L.shared_w : L.wbase + uint64_t(it.slot) * L.wstride;
    const uint32_t mb = q4_matrix_bytes(I, d);
    const uint8_t *qrows[NM];
    const uint16_t *sp[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
        const uint8_t *mat = base + (m / R) * mb;
        const int row = i0 + 16 * (m % R);
        qrows[m] = mat + int64_t(row) * (d / 2) + 16 * bq;
        sp[m] = reinterpret_cast<const uint16_t *>(mat + int64_t(I) * (d / 2)) + int64_t(row + r) * nblk + bq;
    }
    const int tr = min(r, n - 1);
    const int64_t xrow = one ? 0 : sh ? int64_t(it.row0 + tr) : int64_t(L.perm[it.row0 + tr]);
    const uint16_t *xp = reinterpret_cast<const uint16_t *>(L.x) + xrow * d + 8 * g + 32 * bq;
    Rows wr[NM];
    uint32_t sc[NM][CH / 2];
    auto issue = [&](int c0) {
#pragma unroll
        for (int m = 0; m < NM; ++m)
            wr[m].load(qrows[m] + 16 * c0, d / 2, lane);
        if (!(one && c0 == 0)) {
#pragma unroll
            for (int u = 0; u < CH; ++u)
                xv[u] = *reinterpret_cast<const u32x4 *>(xp + 32 * (c0 + u));
        }
#pragma unroll
        for (int m = 0; m < NM; ++m)
            load_scales<CH>(sc[m], sp[m] + c0);
    };
    f32x4 acc[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m)
        acc[m] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int c0 = 0; c0 < nq; c0 += CH) {
        issue(c0);
#pragma unroll
        for (int m = 0; m < NM; ++m)
            wr[m].store(wst[wave] + m * 16 * Rows::RS, lane);
        const uint8_t *q = wst[wave] + r * Rows::RS + 4 * g;
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const bf16x8 xb = as_bf16x8(xv[u]);
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                const uint32_t w = *reinterpret_cast<const uint32_t *>(q + m * 16 * Rows::RS + 16 * u);
                const f32x4 part = mfma16(xb, unpack_q4_16th(w), f32x4{0.f, 0.f, 0.f, 0.f});
                const float s = scale_at(sc[m], u);
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    acc[m][k] = fmaf(s, part[k], acc[m][k]);
            }
        }
    }
    // quarters of d added in wavefront order (a wavefront's LDS operations execute in order, so its sums may take
    // the place of its rows)
    f32x4 *red = reinterpret_cast<f32x4 *>(wst[wave]);
    if (wave > 0) {
#pragma unroll
        for (int m = 0; m < NM; ++m)
            red[m * 64 + lane] = acc[m];
    }
    __syncthreads();
    if (wave != 0 || !slot_gen_ok(it, gnow, L.status))
        return;
#pragma unroll
    for (int w = 1; w < q4s::WAVES; ++w)
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            const f32x4 v = reinterpret_cast<const f32x4 *>(wst[w])[m * 64 + lane];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                acc[m][k] += v[k];
        }
    uint16_t *act = reinterpret_cast<uint16_t *>(sh ? L.act_s : L.act) + int64_t(it.row0) * I + i0 + r;
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int m = 0; m < R; ++m)
            if (4 * g + k < n)
                act[int64_t(4 * g + k) * I + 16 * m] =
                    f32_to_bf16(silu(16.0f * acc[m][k]) * (16.0f * acc[m + R][k]));
}
};

template <int CH, int R>
__global__ void __launch_bounds__(256, 2) stream_gateup_q4_kernel(ExpertLaunch L)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[Q4StreamGateUp<CH, R>::LDS];
    Q4StreamGateUp<CH, R>::run(L, int(blockIdx.x), int(gridDim.x), lds);
}

// Down, 4-bit stream path: a workgroup owns 64 R output columns (16 R per
// wavefront) over all of I, in chunks of CH blocks whose nibbles (through
// WaveRows), act fragments and this lane's block scales are issued together.
// Act rows are the A operand, read straight from global memory (lanes past
// the item's rows repeat its last row), and weights the B operand (outputs:
// tokens 4g .. 4g + 3 of columns c0 + 16 m + r).
template <int CH, int R>
struct Q4StreamDown {
using Rows = WaveRows<16 * CH>;
static constexpr int REGION = R * 16 * Rows::RS;
static constexpr size_t LDS = q4s::WAVES * REGION;
static constexpr int WAVES_PER_SIMD = 4;
static __device__ __forceinline__ void run(const ExpertLaunch &L, int block, int n_blocks, uint8_t *lds)
{
    uint8_t (*wst)[REGION] = reinterpret_cast<uint8_t (*)[REGION]>(lds);
    int t;
    WorkItem it;
    if (!q4_tile(L, L.d / (q4s::WAVES * q4s::ROWS * R), block, n_blocks, t, it) || it.nrows == 0)   // nrows 0: unpublished expert
        return;
    // the generation is read here and compared before the stores, and the row weights are read with the
    // first weights, so nothing waits between the item lookup and the weight loads
    const uint32_t gnow = slot_gen_now(it, L.gen_dev);
    const int n = it.nrows, d = L.d, I = L.I, nblk = I / 32;
    const bool sh = it.slot < 0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c0 = ((t - it.tile0) * q4s::WAVES + wave) * q4s::ROWS * R;
    const int r = lane & 15, g = lane >> 4;
    const uint8_t *base = sh ? L.shared_w : L.wbase + uint64_t(it.slot) * L.wstride;
    const uint8_t *wd = base + 2 * q4_matrix_bytes(I, d);
    const uint8_t *qrows = wd + int64_t(c0) * (I / 2);
    const uint16_t *sp = reinterpret_cast<const uint16_t *>(wd + int64_t(d) * (I / 2)) + int64_t(c0 + r) * nblk;
    const uint16_t *ap = reinterpret_cast<const uint16_t *>(sh ? L.act_s : L.act) +
                         int64_t(it.row0 + min(r, n - 1)) * I + 8 * g;
    Rows wr[R];
    u32x4 av[CH];
    uint32_t sc[R][CH / 2];
    f32x4 acc[R];
#pragma unroll
    for (int m = 0; m < R; ++m)
        acc[m] = f32x4{0.f, 0.f, 0.f, 0.f};
    float rw[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        rw[k] = (sh || 4 * g + k >= n) ? 1.0f : L.row_weight[it.row0 + 4 * g + k];
    for (int b0 = 0; b0 < nblk; b0 += CH) {
#pragma unroll
        for (int m = 0; m < R; ++m)
            wr[m].load(qrows + int64_t(16 * m) * (I / 2) + 16 * b0, I / 2, lane);
#pragma unroll
        for (int u = 0; u < CH; ++u)
            av[u] = *reinterpret_cast<const u32x4 *>(ap + 32 * (b0 + u));
#pragma unroll
        for (int m = 0; m < R; ++m)
            load_scales<CH>(sc[m], sp + int64_t(16 * m) * nblk + b0);
#pragma unroll
        for (int m = 0; m < R; ++m)
            wr[m].store(wst[wave] + m * 16 * Rows::RS, lane);
        const uint8_t *q = wst[wave] + r * Rows::RS + 4 * g;
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const bf16x8 ab = as_bf16x8(av[u]);
#pragma unroll
            for (int m = 0; m < R; ++m) {
                const uint32_t w = *reinterpret_cast<const uint32_t *>(q + m * 16 * Rows::RS + 16 * u);
                const f32x4 part = mfma16(ab, unpack_q4_16th(w), f32x4{0.f, 0.f, 0.f, 0.f});
                const float sv = scale_at(sc[m], u);
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    acc[m][k] = fmaf(sv, part[k], acc[m][k]);
            }
        }
    }
    if (!slot_gen_ok(it, gnow, L.status))
        return;
    uint16_t *y = static_cast<uint16_t *>(sh ? L.ys : L.y) + int64_t(it.row0) * d + c0 + r;
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int m = 0; m < R; ++m)
            if (4 * g + k < n)
                y[int64_t(4 * g + k) * d + 16 * m] = f32_to_bf16((16.0f * acc[m][k]) * rw[k]);
}
};

template <int CH, int R>
__global__ void __launch_bounds__(256, 2) stream_down_q4_kernel(ExpertLaunch L)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[Q4StreamDown<CH, R>::LDS];
    Q4StreamDown<CH, R>::run(L, int(blockIdx.x), int(gridDim.x), lds);
}

template <int R>
static int tiles_gateup_q4_stream(int, int, int I)
{
    return I / (q4s::ROWS * R);
}

template <int R>
static int tiles_down_q4_stream(int, int d, int)
{
    return d / (q4s::WAVES * q4s::ROWS * R);
}

template <int R>
static hipError_t launch_gateup_q4_stream(const ExpertLaunch &L, hipStream_t s)
{
    if (L.n_tiles == 0)
        return hipSuccess;
    // chunk: the largest of 8, 4, 2 blocks dividing a quarter of d (d % 256 == 0)
    const int nq = L.d / 128;
    if (nq % 8 == 0)
        launch_k(stream_gateup_q4_kernel<8, R>, L.n_tiles, 256, 0, s, L);
    else if (nq % 4 == 0)
        launch_k(stream_gateup_q4_kernel<4, R>, L.n_tiles, 256, 0, s, L);
    else
        launch_k(stream_gateup_q4_kernel<2, R>, L.n_tiles, 256, 0, s, L);
    return hipGetLastError();
}

template <int R>
static hipError_t launch_down_q4_stream(const ExpertLaunch &L, hipStream_t s)
{
    if (L.n_tiles == 0)
        return hipSuccess;
    // chunk: 8 or 4 blocks dividing I / 32 (I % 128 == 0)
    if (L.I % 256 == 0)
        launch_k(stream_down_q4_kernel<8, R>, L.n_tiles, 256, 0, s, L);
    else
        launch_k(stream_down_q4_kernel<4, R>, L.n_tiles, 256, 0, s, L);
    return hipGetLastError();
}

// ============================================================== tile path

namespace q4t {
constexpr int BK = 64, ROWB = BK * 2, QROWB = BK / 2;   // K elements per stage; bytes of a staged row of A, of codes

template <bool GU_, int BM_, int TN_, int WR_, int WC_, int WPC_>
struct Shape {
    static constexpr bool GU = GU_;
    static constexpr int BM = BM_, TN = TN_, WR = WR_, WC = WC_, WPC = WPC_;   // rows, weight rows, wavefronts, per CU
    static constexpr int WAVES = WR * WC, THREADS = 64 * WAVES;
    static constexpr int MB = BM / WR / 16, NB = TN / WC / 16;
    static constexpr int A_BYTES = BM * ROWB, Q_BYTES = TN * QROWB, S_BYTES = TN * 4;
    static constexpr int STAGE = A_BYTES + Q_BYTES + S_BYTES;
    static constexpr int LA = BM / 8 / WAVES, LQ = TN / 32 / WAVES, NS = TN / 64;
    static constexpr size_t LDS = size_t(2) * STAGE;
    static_assert(BM % (8 * WAVES) == 0 && TN % (32 * WAVES) == 0 && NS <= WAVES && LDS * WPC <= 160 * 1024, "");
};
}  // namespace q4t

// Gate/up: tile columns 0 .. TN/2 - 1 are gate rows nt TN/2 .., the rest the
// matching up rows; wavefront (wm, wn) owns MB 16-row blocks and NB column
// blocks (gate/up: NB / 2 gate blocks and the matching up blocks, so SiLU * up
// forms in registers).  Weights are the A operand: a lane's outputs are
// columns 4g .. 4g + 3 of row r16, stored as 16-byte pieces straight to memory.
// Stages go from memory straight into two LDS buffers (buffer loads with an
// LDS destination), one ahead: rows of A as eight 16-byte chunks, chunk c of
// row r in slot c ^ ((r / 2) % 8), codes as two chunks, chunk c of row r in slot
// c ^ ((r / 8) % 2), which puts the 16 rows of each fragment read on distinct
// banks, and the rows' two scales.  The codes enter the MFMA as 136 + q; the
// -136 * (block sum of the token row) that takes the offset back out comes from
// one more MFMA per token fragment, against a fragment of -136, and is the C
// input of that fragment's block partials.
template <class S>
struct Q4Tile {
static constexpr size_t LDS = S::LDS;
static constexpr int WAVES_PER_SIMD = S::WPC * S::WAVES / 4;
static __device__ __forceinline__ void run(const ExpertLaunch &L, int block, int n_blocks, uint8_t *lds8)
{
    using namespace q4t;
    constexpr bool GU = S::GU;
    constexpr int BM = S::BM, TN = S::TN, WAVES = S::WAVES, MB = S::MB, NB = S::NB, STAGE = S::STAGE;
    int n_items, n_tiles;
    const int t = launch_tile(L, block, n_blocks, n_items, n_tiles);
    if (t < 0)
        return;                                   // past the device-built list's tiles
    const WorkItem it = L.items[find_item(L.items, n_items, t)];
    const uint32_t gnow = slot_gen_now(it, L.gen_dev);   // compared before the stores
    const bool sh = it.slot < 0;
    const int d = L.d, I = L.I;
    const int K = GU ? d : I;
    const int ntn = GU ? I / (TN / 2) : d / TN;
    const int local = t - it.tile0;
    const int m0 = (local / ntn) * BM;
    const int nt = local % ntn;
    const int valid = min(BM, it.nrows - m0);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // (uniform: copy destinations and resources)
    const int wm = wave / S::WC, wn = wave % S::WC;
    const int r16 = lane & 15, g = lane >> 4;

    const uint8_t *obj = sh ? L.shared_w : L.wbase + uint64_t(it.slot) * L.wstride;
    const uint32_t mbytes = q4_matrix_bytes(I, d);
    // byte offset, from the object, of tile column c's matrix and its row there
    auto col_matrix = [&](int c) -> uint32_t { return GU ? (c < TN / 2 ? 0u : mbytes) : 2 * mbytes; };
    auto col_row = [&](int c) -> uint32_t {
        return GU ? uint32_t(nt * (TN / 2) + (c < TN / 2 ? c : c - TN / 2)) : uint32_t(nt * TN + c);
    };
    [[maybe_unused]] const void *abase = GU ? L.x
                                            : static_cast<const uint8_t *>(sh ? L.act_s : L.act) +
                                                  (int64_t(it.row0) + m0) * int64_t(I) * 2;
    uint32_t aoff[S::LA], qoff[S::LQ];
#pragma unroll
    for (int i = 0; i < S::LA; ++i) {
        const int r = 8 * (WAVES * i + wave) + (lane >> 3);
        const int m = m0 + min(r, valid - 1);     // rows past the end repeat the last one and are never stored
        const uint32_t src = !GU ? uint32_t(m - m0) : sh ? uint32_t(it.row0 + m) : uint32_t(L.perm[it.row0 + m]);
        aoff[i] = src * uint32_t(K * 2) + uint32_t(((lane & 7) ^ ((r >> 1) & 7)) << 4);
    }
#pragma unroll
    for (int i = 0; i < S::LQ; ++i) {
        const int c = 32 * (WAVES * i + wave) + (lane >> 1);
        qoff[i] = col_matrix(c) + col_row(c) * uint32_t(K / 2) + uint32_t(16 * ((lane & 1) ^ ((c >> 3) & 1)));
    }
    const int sc_col = 64 * (wave % S::NS) + lane;
    [[maybe_unused]] const uint32_t soff = col_matrix(sc_col) + uint32_t(GU ? I : d) * uint32_t(K / 2) +
                                           col_row(sc_col) * uint32_t(K / 32) * 2u;
    auto issue = [&](int stage, int buf) {
        uint8_t *st = lds8 + buf * STAGE;
#if defined(__HIP_DEVICE_COMPILE__)
        const __amdgpu_buffer_rsrc_t ar =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(abase), 0, 0x7fffffff, 0x00020000u);
        const __amdgpu_buffer_rsrc_t wr_ =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(obj), 0, 0x7fffffff, 0x00020000u);
#pragma unroll
        for (int i = 0; i < S::LA; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ar, (lds_void_t *)(st + (WAVES * i + wave) * 1024), 16, aoff[i],
                                                     stage * ROWB, 0, 0);
#pragma unroll
        for (int i = 0; i < S::LQ; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr_, (lds_void_t *)(st + S::A_BYTES + (WAVES * i + wave) * 1024),
                                                     16, qoff[i], stage * QROWB, 0, 0);
        if (wave < S::NS)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr_, (lds_void_t *)(st + S::A_BYTES + S::Q_BYTES + wave * 256), 4,
                                                     soff, stage * 4, 0, 0);
#else
        (void)st, (void)stage;
#endif
    };

    auto col_of = [&](int nb) -> int {              // tile column block of this wavefront
        if (GU)
            return nb < NB / 2 ? (wn * (NB / 2) + nb) * 16 : TN / 2 + (wn * (NB / 2) + nb - NB / 2) * 16;
        return (wn * NB + nb) * 16;
    };
    f32x4 acc[NB][MB];
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int b = 0; b < MB; ++b)
            acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bf16x8 neg136 = __builtin_bit_cast(bf16x8, u32x4{0xC308C308u, 0xC308C308u, 0xC308C308u, 0xC308C308u});
    auto compute = [&](int buf) {
        const uint8_t *st = lds8 + buf * STAGE;
#pragma unroll
        for (int kb = 0; kb < BK / 32; ++kb) {
            uint32_t cw[NB];
            u32x4 sc[NB];                           // the scales of rows 4g .. 4g + 3, both blocks
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const int c = col_of(nb) + r16;                    // A fragment: weight row c
                cw[nb] = *reinterpret_cast<const uint32_t *>(st + S::A_BYTES + c * QROWB + 16 * (kb ^ ((c >> 3) & 1)) +
                                                             4 * g);
                sc[nb] = *reinterpret_cast<const u32x4 *>(st + S::A_BYTES + S::Q_BYTES + (col_of(nb) + 4 * g) * 4);
            }
            bf16x8 af[MB];
            f32x4 corr[MB];
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                const int r = (wm * MB + mb) * 16 + r16;
                af[mb] = as_bf16x8(*reinterpret_cast<const u32x4 *>(st + r * ROWB + (((4 * kb + g) ^ ((r >> 1) & 7)) << 4)));
                corr[mb] = mfma16(neg136, af[mb], f32x4{0.f, 0.f, 0.f, 0.f});
            }
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const bf16x8 w = unpack_q4_136(cw[nb]);
                f32x4 part[MB];
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
                    part[mb] = mfma16(w, af[mb], corr[mb]);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float s = half_to_float(uint16_t(sc[nb][i] >> (16 * kb)));
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb)
                        acc[nb][mb][i] = fmaf(s, part[mb][i], acc[nb][mb][i]);
                }
            }
        }
    };

    const int nk = K / BK;
    issue(0, 0);
    for (int kt = 0; kt < nk; ++kt) {
        __builtin_amdgcn_s_waitcnt(VMCNT_WAIT(0));  // this stage landed ...
        __builtin_amdgcn_s_barrier();               // ... for every wavefront; the other buffer was last read
        asm volatile("" ::: "memory");              //     one stage ago
        if (kt + 1 < nk)
            issue(kt + 1, (kt + 1) & 1);
        compute(kt & 1);
    }
    if (!slot_gen_ok(it, gnow, L.status))
        return;

    // ---- epilogue: lane holds columns 4g .. 4g + 3 of each block of row r16; two blocks at a time are regrouped
    // so that each lane stores 16 contiguous bytes
    const int64_t rowbase = int64_t(it.row0) + m0;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        const int row = (wm * MB + mb) * 16 + r16;
        const bool in = row < valid;
        constexpr int OB = GU ? NB / 2 : NB;        // output blocks
        uint32_t lo[OB], hi[OB];
        if constexpr (GU) {
#pragma unroll
            for (int nb = 0; nb < OB; ++nb) {
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    v[i] = silu(acc[nb][mb][i]) * acc[nb + OB][mb][i];
                lo[nb] = pack_bf16x2_hw(v[0], v[1]);
                hi[nb] = pack_bf16x2_hw(v[2], v[3]);
            }
        } else {
            const float w = (sh || !in) ? 1.0f : L.row_weight[rowbase + row];
#pragma unroll
            for (int nb = 0; nb < OB; ++nb) {
                lo[nb] = pack_bf16x2_hw(acc[nb][mb][0] * w, acc[nb][mb][1] * w);
                hi[nb] = pack_bf16x2_hw(acc[nb][mb][2] * w, acc[nb][mb][3] * w);
            }
        }
        uint16_t *dst = GU ? static_cast<uint16_t *>(sh ? L.act_s : L.act) + (rowbase + row) * I + nt * (TN / 2)
                           : static_cast<uint16_t *>(sh ? L.ys : L.y) + (rowbase + row) * d + nt * TN;
        dst += wn * OB * 16;
        if constexpr (OB == 1) {
            if (in)
                *reinterpret_cast<uint2 *>(dst + 4 * g) = make_uint2(lo[0], hi[0]);
        } else {
#pragma unroll
            for (int k = 0; k < OB / 2; ++k) {
                const uint4 v = gather16(lo[2 * k], hi[2 * k], lo[2 * k + 1], hi[2 * k + 1]);
                if (in)
                    *reinterpret_cast<uint4 *>(dst + 32 * k + 8 * g) = v;
            }
        }
    }
}
};

template <class S>
__global__ void __launch_bounds__(S::THREADS, S::WPC *S::WAVES / 4) tile_q4_kernel(ExpertLaunch L)
{
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds8[];
    Q4Tile<S>::run(L, int(blockIdx.x), int(gridDim.x), lds8);
}

template <class S>
static int q4_tiles(int nrows, int d, int I)
{
    return (nrows + S::BM - 1) / S::BM * (S::GU ? I / (S::TN / 2) : d / S::TN);
}

template <class S>
static TileGeom q4_geom(int d, int I)
{
    return TileGeom{S::BM, S::GU ? I / (S::TN / 2) : d / S::TN};
}

template <class S>
static hipError_t launch_q4_tile(const ExpertLaunch &L, hipStream_t s)
{
    if (L.n_tiles == 0)
        return hipSuccess;
    launch_k(tile_q4_kernel<S>, L.n_tiles, S::THREADS, S::LDS, s, L);
    return hipGetLastError();
}

using Q4GateSmall = q4t::Shape<true, 64, 128, 1, 4, 4>;
using Q4GateBig = q4t::Shape<true, 128, 128, 2, 2, 2>;
using Q4Down = q4t::Shape<false, 64, 128, 1, 2, 6>;

// The 64-row gate/up tiles, or the down tiles, and the stream list in one
// launch (both_kernel).  Measured (MI355X, E 512, d 2048, I 512, K 10, router
// bias 0.3 ln Zipf(1.5); gate/up, us): two launches 25 + 79 (128 tokens),
// 47 + 110 (509), 99 + 112 (1013); together 81, 141, 189; down 15 + 43,
// 25 + 60, 50 + 62 and 52, 88, 115 (the two launches without the gap between
// them).  The down tiles take four workgroups per CU here, not six, which is
// what the stream list's registers allow.
using Q4DownBoth = q4t::Shape<false, 64, 128, 1, 4, 4>;

static hipError_t launch_gateup_q4_both(const ExpertLaunch &T, const ExpertLaunch &S, hipStream_t s)
{
    const int nq = S.d / 128;
    if (nq % 8 == 0)
        return launch_both<Q4Tile<Q4GateSmall>, Q4StreamGateUp<8, 2>>(T, S, s);
    if (nq % 4 == 0)
        return launch_both<Q4Tile<Q4GateSmall>, Q4StreamGateUp<4, 2>>(T, S, s);
    return launch_both<Q4Tile<Q4GateSmall>, Q4StreamGateUp<2, 2>>(T, S, s);
}

static hipError_t launch_down_q4_both(const ExpertLaunch &T, const ExpertLaunch &S, hipStream_t s)
{
    if (S.I % 256 == 0)
        return launch_both<Q4Tile<Q4DownBoth>, Q4StreamDown<8, 2>>(T, S, s);
    return launch_both<Q4Tile<Q4DownBoth>, Q4StreamDown<4, 2>>(T, S, s);
}

template <class G, int R>
static const KernelSet q4_set{q4_tiles<G>, tiles_gateup_q4_stream<R>, q4_tiles<Q4Down>, tiles_down_q4_stream<R>,
                              q4_geom<G>, q4_geom<Q4Down>,
                              launch_q4_tile<G>, launch_gateup_q4_stream<R>,
                              launch_q4_tile<Q4Down>, launch_down_q4_stream<R>,
                              R == 2 && G::BM == 64 ? launch_gateup_q4_both : nullptr,
                              R == 2 && G::BM == 64 ? launch_down_q4_both : nullptr};

// Tile forms by the mean rows per expert, R of the stream kernels by what
// bounds the launch's items: the experts and routed rows of a decode, the
// largest round on the scheduled path; on the device-built lists of more than
// 16 tokens the routed rows alone (the joint launches are R = 2).  From 32 on
// R = 2; fewer items leave CUs idle with it: E 128, K 4, 16 tokens, 48 slots,
// d 1024, I 768 318 us a step, 329 with R = 2; E 8, K 2, d 2048, I 4096 resident
// 88 against 96.  All forms are
// bit-identical (the same chain of operations per output), so the choice is
// the launch's.  Measured (MI355X, E 512, d 2048, I 512, K 10, us):
//   router bias 0.3 ln Zipf(1.5), stream gate/up + down, R = 1, R = 2: T 1
//   8.2+5.2, 9.8+6.5; T 2 9.5+6.7, 12+7.8; T 4 13.3+9.4, 15+10; T 6 17+10.5,
//   15.6+10.4; T 8 19.6+12.6, 21.8+11.6; T 16 27.5+18.4, 28.6+17.0; T 1013
//   111+78, 112+62, and gate/up in one launch with the tiles 208, 189;
//   no bias, tile gate/up 64 x 128, 128 x 128: mean rows 20 199, 304; 40 278,
//   403; 80 447, 409; 640 2465, 2327; down 64 x 128 by two wavefronts 40 127, 80
//   220, 640 1190 (128 x 128, a form no longer here: 223, 241, 1407).
const KernelSet &q4_kernels(uint64_t rows, uint64_t E, uint64_t items)
{
    if (items < 32 && rows <= 64 * E)
        return q4_set<Q4GateSmall, 1>;
    return rows <= 64 * E ? q4_set<Q4GateSmall, 2> : q4_set<Q4GateBig, 2>;
}

hipError_t init_q4_attributes()
{
    for (const void *k : {reinterpret_cast<const void *>(&tile_q4_kernel<Q4GateSmall>),
                          reinterpret_cast<const void *>(&tile_q4_kernel<Q4GateBig>),
                          reinterpret_cast<const void *>(&tile_q4_kernel<Q4Down>)}) {
        const hipError_t e = allow_large_lds(k);
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

}  // namespace msi
