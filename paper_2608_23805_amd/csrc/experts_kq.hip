// experts_kq.hip -- expert projections of the quantized-expert mix (the
// paper's 4.5 / 6.5625 bits-per-weight representation, "Implementation" and
// "Output-Exact Execution Beyond the Full-Residency Envelope"), gfx950.
//
// Formats (per matrix [rows, cols], 256-element super-blocks along a row):
//  * k4 (Wg, Wu): nibbles [rows, cols/2] (unsigned 0..15, element 2j in the
//    low nibble of byte j), then a 16-byte header per (row, super-block):
//    fp16 d, fp16 dmin, eight 6-bit sub-block scales, eight 6-bit sub-block
//    mins (48-bit little-endian fields); value = d sc_j q - dmin m_j for the
//    j-th 32-element sub-block.
//  * k6 (Wd): low nibbles [rows, cols/2], high 2-bit parts [rows, cols/4]
//    (element 4j + t at bits 2t of byte j), int8 scales [rows, cols/16], fp16
//    d [rows, cols/256]; q = low | high << 4 and value = d sc_j (q - 32) for
//    the j-th 16-element sub-block.
//
// The stream path applies each sub-block's scale in fp32: the k6 integers
// q - 32 and the k4 integers 128 + q are exact in bf16, so every MFMA partial
// over a sub-block is a sum of exact products.  The k4 min term takes the
// tokens' sums over the sub-block (one more MFMA, against a fragment of ones)
// times dmin m_j + 128 d sc_j, which also removes the 128 of the operands.  A
// 16x16x32 MFMA spans one k4 sub-block, or two k6 sub-blocks: those are split
// by zeroing the weight lanes of the other half (lanes 0..31 carry elements
// 0..15 of the 32).
//
//  * stream path (<= 16 tokens per expert): tokens as the A operand, read
//    straight from memory, and weights as the B operand (WaveRows), so each
//    output lane holds one weight row (and that row's coefficients) for four
//    tokens;
//  * tile path: 64 x 128 or 128 x 256 outputs per workgroup, whole
//    super-blocks summed in units of their d (described there).
#include "common.h"
#include "gemm_ring.h"
#include "kernels.h"

namespace msi {

namespace {

constexpr uint32_t BF16_ONE2 = 0x3F803F80u;        // two bf16 1.0

__device__ __forceinline__ float h2f(uint16_t h) { return float(__builtin_bit_cast(_Float16, h)); }
__device__ __forceinline__ uint16_t f16_bits(float f) { return __builtin_bit_cast(uint16_t, _Float16(f)); }

// 8 k6 elements: low nibbles (element e at bits 4e of lo) and 2-bit high
// parts (element e at bits 2e of hi) -> 8 exact bf16 values q - 32.  The
// codes are assembled one per byte (even and odd elements in two words), each
// byte converted to binary32 by the byte-to-float instructions and 32
// subtracted: q - 32 exactly, and that integer (at most 6 significant bits) is
// exact in the top half of its binary32.
__device__ __forceinline__ bf16x8 unpack_k6(uint32_t lo, uint32_t hi)
{
    // spread the four 4-bit groups of hi (two elements each) to bytes 0..3
    uint32_t t = (hi | (hi << 8)) & 0x00FF00FFu;
    t = (t | (t << 4)) & 0x0F0F0F0Fu;
    const uint32_t ev = (lo & 0x0F0F0F0Fu) | ((t & 0x03030303u) << 4);          // elements 0, 2, 4, 6
    const uint32_t od = ((lo >> 4) & 0x0F0F0F0Fu) | ((t & 0x0C0C0C0Cu) << 2);   // elements 1, 3, 5, 7
    u32x4 r;
    float c32 = 32.0f;
    asm("" : "+v"(c32));        // (kept a register: the byte conversions then stay v_cvt_f32_ubyte)
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const float fe = float((ev >> (8 * h)) & 0xFFu) - c32;
        const float fo = float((od >> (8 * h)) & 0xFFu) - c32;
        r[h] = __builtin_amdgcn_perm(__float_as_uint(fo), __float_as_uint(fe), 0x07060302u);
    }
    return __builtin_bit_cast(bf16x8, r);
}

// k4 header (16 bytes as four words): sub-block j's scale d sc_j and offset dmin m_j
__device__ __forceinline__ void k4_coef(const u32x4 &h, int j, float &a, float &b)
{
    const uint64_t sc = uint64_t(h[1]) | (uint64_t(h[2] & 0xFFFFu) << 32);
    const uint64_t mn = uint64_t(h[2] >> 16) | (uint64_t(h[3]) << 16);
    a = h2f(uint16_t(h[0])) * float(uint32_t(sc >> (6 * j)) & 63u);
    b = h2f(uint16_t(h[0] >> 16)) * float(uint32_t(mn >> (6 * j)) & 63u);
}

// the same with the min coefficient taken against partials over 128 + q:
// a (P + 128 S) - (b + 128 a) S = a P - b S
__device__ __forceinline__ void k4_coef128(const u32x4 &h, int j, float &a, float &b)
{
    k4_coef(h, j, a, b);
    b = fmaf(128.0f, a, b);
}

__host__ __device__ __forceinline__ uint32_t k4_bytes(uint32_t rows, uint32_t cols)
{
    return rows * (cols / 2) + rows * (cols / 256) * 16u;
}

// k6 planes of a [rows, cols] matrix at m: low nibbles, high parts, scales, d
struct K6Planes {
    const uint8_t *ql, *qh;
    const int8_t *sc;
    const uint16_t *d;
};
__device__ __forceinline__ K6Planes k6_planes(const uint8_t *m, uint32_t rows, uint32_t cols)
{
    K6Planes p;
    p.ql = m;
    p.qh = m + rows * (cols / 2);
    p.sc = reinterpret_cast<const int8_t *>(p.qh + rows * (cols / 4));
    p.d = reinterpret_cast<const uint16_t *>(reinterpret_cast<const uint8_t *>(p.sc) + rows * (cols / 16));
    return p;
}

// Tile of a launch and its item (device-built decode list, device-built
// prefill list, or host list), as the 4-bit kernels find theirs.
__device__ __forceinline__ bool kq_tile(const ExpertLaunch &L, int per_item, int b, int n_blocks, int &t, WorkItem &it)
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

}  // namespace

// ============================================================== stream path

namespace kqs {
constexpr int WAVES = 4, ROWS = 16;
}

// Gate/up, k4 stream path: a workgroup owns 16 R rows of Wg and of Wu; its
// four wavefronts take the quarters of d and add their partial sums in
// wavefront order.  Tokens are the A operand and weights the B operand, so
// lane (r = lane % 16, g = lane / 16) holds elements 8g .. 8g + 7 of each block
// of token r and of weight rows i0 + 16 m + r, and its outputs are tokens
// 4g .. 4g + 3 of those rows: one row's sub-block coefficients per lane and
// row group.  Token fragments come straight from global memory (the few rows
// of a decode step stay in cache; lanes past the item's rows repeat its last
// row and are not stored); weights go through WaveRows.  Blocks go in chunks
// of CH (CH divides 8: at most one super-block), each chunk's loads issued
// before its first MFMA.  The four lanes of a weight row share the decoding of
// its sub-block coefficients: lane (r, g) decodes those of blocks g, g + 4 of
// the chunk into the wavefront's LDS table, and every lane reads the block's
// coefficients back.  R = 2 where a launch has many items: a token fragment
// (1 KiB from 16 rows) then serves twice the codes (see the 4-bit kernels).
template <int CH, int R>
struct KqStreamGateUp {
using Rows = WaveRows<16 * CH>;
static constexpr int NM = 2 * R;                       // 16-row groups: R of Wg, then R of Wu
static constexpr int REGION = NM * 16 * Rows::RS > NM * 1024 ? NM * 16 * Rows::RS : NM * 1024;
static constexpr size_t LDS = kqs::WAVES * (REGION + CH * NM * 16 * sizeof(float2));
static constexpr int WAVES_PER_SIMD = 3;
static __device__ __forceinline__ void run(const ExpertLaunch &L, int block, int n_blocks, uint8_t *lds)
{
    // a wavefront's rows, then (its own part) its partial sums; {a, b} of block u, row group m, row r
    uint8_t (*wst)[REGION] = reinterpret_cast<uint8_t (*)[REGION]>(lds);
    float2 (*coef)[CH][NM][16] = reinterpret_cast<float2 (*)[CH][NM][16]>(lds + kqs::WAVES * REGION);
    int t;
    WorkItem it;
    if (!kq_tile(L, L.I / (kqs::ROWS * R), block, n_blocks, t, it) || it.nrows == 0 ||
        !slot_current(it, L.gen_dev, L.status))      // nrows 0: unpublished expert, no work
        return;
    static_assert(CH <= 8, "a chunk stays within one super-block");
    const int n = it.nrows, d = L.d, I = L.I, nsb = d / 256, nq = d / 32 / kqs::WAVES;
    const bool sh = it.slot < 0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i0 = (t - it.tile0) * kqs::ROWS * R;
    const int r = lane & 15, g = lane >> 4;
    const int bq = wave * nq;                          // this wavefront's first block
    const uint8_t *base = sh ? L.shared_w : L.wbase + uint64_t(it.slot) * L.wstride;
    const uint32_t mb = k4_bytes(I, d);
    const uint8_t *qrows[NM];
    const u32x4 *hp[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
        const uint8_t *mat = base + (m / R) * mb;
        const int row = i0 + 16 * (m % R);
        qrows[m] = mat + int64_t(row) * (d / 2) + 16 * bq;
        hp[m] = reinterpret_cast<const u32x4 *>(mat + uint32_t(I) * uint32_t(d / 2)) + int64_t(row + r) * nsb;
    }
    const int tr = min(r, n - 1);
    const int64_t xrow = sh ? int64_t(it.row0 + tr) : int64_t(L.perm[it.row0 + tr]);
    const uint16_t *xp = reinterpret_cast<const uint16_t *>(L.x) + xrow * d + 8 * g + 32 * bq;
    Rows wr[NM];
    u32x4 xv[CH], hd[NM];                              // token fragments; the chunk's super-block headers
    auto issue = [&](int c0) {
#pragma unroll
        for (int m = 0; m < NM; ++m)
            wr[m].load(qrows[m] + 16 * c0, d / 2, lane);
#pragma unroll
        for (int u = 0; u < CH; ++u)
            xv[u] = *reinterpret_cast<const u32x4 *>(xp + 32 * (c0 + u));
#pragma unroll
        for (int m = 0; m < NM; ++m)
            hd[m] = hp[m][(bq + c0) >> 3];
    };
    const bf16x8 ones = __builtin_bit_cast(bf16x8, u32x4{BF16_ONE2, BF16_ONE2, BF16_ONE2, BF16_ONE2});
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
        for (int u0 = 0; u0 < CH; u0 += 4) {
            const int u = u0 + g;
            if (u < CH) {
                const int j = (bq + c0 + u) & 7;       // sub-block within the super-block
#pragma unroll
                for (int m = 0; m < NM; ++m) {
                    float a, b;
                    k4_coef128(hd[m], j, a, b);
                    coef[wave][u][m][r] = make_float2(a, b);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const bf16x8 xb = pair_order(xv[u]);
            const f32x4 sx = mfma16(xb, ones, f32x4{0.f, 0.f, 0.f, 0.f});    // the tokens' sums over the block
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                const f32x4 part =
                    mfma16(xb, unpack_u4_pairs(*reinterpret_cast<const uint32_t *>(q + m * 16 * Rows::RS + 16 * u)),
                           f32x4{0.f, 0.f, 0.f, 0.f});
                const float2 cf = coef[wave][u][m][r];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    acc[m][i] = fmaf(cf.x, part[i], acc[m][i]);
                    acc[m][i] = fmaf(-cf.y, sx[i], acc[m][i]);
                }
            }
        }
    }
    // quarters of d added in wavefront order (a wavefront's LDS operations execute in order, so its sums may take
    // the place of its rows)
    if (wave > 0) {
        f32x4 *red = reinterpret_cast<f32x4 *>(wst[wave]);
#pragma unroll
        for (int m = 0; m < NM; ++m)
            red[m * 64 + lane] = acc[m];
    }
    __syncthreads();
    if (wave != 0)
        return;
#pragma unroll
    for (int w = 1; w < kqs::WAVES; ++w)
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            const f32x4 v = reinterpret_cast<const f32x4 *>(wst[w])[m * 64 + lane];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                acc[m][i] += v[i];
        }
    uint16_t *act = reinterpret_cast<uint16_t *>(sh ? L.act_s : L.act) + int64_t(it.row0) * I + i0 + r;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int m = 0; m < R; ++m)
            if (4 * g + i < n)
                act[int64_t(4 * g + i) * I + 16 * m] = f32_to_bf16(silu(acc[m][i]) * acc[m + R][i]);
}
};

template <int CH, int R>
__global__ void __launch_bounds__(256, R == 1 ? 3 : 2) stream_gateup_kq_kernel(ExpertLaunch L)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[KqStreamGateUp<CH, R>::LDS];
    KqStreamGateUp<CH, R>::run(L, int(blockIdx.x), int(gridDim.x), lds);
}

// Down, k6 stream path: a workgroup owns 64 output columns (16 per wavefront)
// over all of I, in groups of G super-blocks whose low nibbles and high parts
// (through WaveRows), act fragments and this lane's sub-block and
// super-block scales are issued together.  Act rows are the A operand, read
// straight from global memory (lanes past the item's rows repeat its last
// row), and weights the B operand (lane: token r / weight row c0 + r,
// elements 8g .. 8g + 7 of each block; outputs: tokens 4g .. 4g + 3 of column
// c0 + r).  Each 32-element block holds two 16-element sub-blocks: two MFMAs
// with the other half's weight lanes zeroed (lanes with g < 2 carry elements
// 0 .. 15), each partial scaled by its own d * sc.
template <int G>
__global__ void __launch_bounds__(256, 2) stream_down_kq_kernel(ExpertLaunch L)
{
    constexpr int NB = 8 * G;                          // 32-element blocks per group
    using QL = WaveRows<16 * NB>;                      // 16 bytes of low nibbles per block
    using QH = WaveRows<8 * NB>;                       // 8 bytes of high parts per block
    __shared__ __attribute__((aligned(16))) uint8_t lst[kqs::WAVES][16 * QL::RS];
    __shared__ __attribute__((aligned(16))) uint8_t hst[kqs::WAVES][16 * QH::RS];
    int t;
    WorkItem it;
    if (!kq_tile(L, L.d / (kqs::WAVES * kqs::ROWS), int(blockIdx.x), int(gridDim.x), t, it) || it.nrows == 0 ||
        !slot_current(it, L.gen_dev, L.status))      // nrows 0: unpublished expert, no work
        return;
    const int n = it.nrows, d = L.d, I = L.I, nsb = I / 256;
    const bool sh = it.slot < 0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c0 = ((t - it.tile0) * kqs::WAVES + wave) * kqs::ROWS;
    const int r = lane & 15, g = lane >> 4;
    const uint8_t *base = sh ? L.shared_w : L.wbase + uint64_t(it.slot) * L.wstride;
    const K6Planes P = k6_planes(base + 2 * k4_bytes(I, d), d, I);
    const int64_t row = c0 + r;                        // this lane's weight row (output column)
    const uint8_t *qlrows = P.ql + int64_t(c0) * (I / 2);
    const uint8_t *qhrows = P.qh + int64_t(c0) * (I / 4);
    const u32x4 *scp = reinterpret_cast<const u32x4 *>(P.sc + row * (I / 16));
    const uint16_t *ap = reinterpret_cast<const uint16_t *>(sh ? L.act_s : L.act) +
                         int64_t(it.row0 + min(r, n - 1)) * I + 8 * g;
    QL wl;
    QH wh;
    u32x4 av[NB], sc[G];
    float dd[G];
    auto issue = [&](int s0) {
        wl.load(qlrows + 128 * s0, I / 2, lane);
        wh.load(qhrows + 64 * s0, I / 4, lane);
#pragma unroll
        for (int u = 0; u < NB; ++u)
            av[u] = *reinterpret_cast<const u32x4 *>(ap + 32 * (8 * s0 + u));
#pragma unroll
        for (int s = 0; s < G; ++s) {
            sc[s] = scp[s0 + s];
            dd[s] = h2f(P.d[row * nsb + s0 + s]);
        }
    };
    const bool first_half = g < 2;
    const bf16x8 zero = __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < nsb; s0 += G) {
        issue(s0);
        wl.store(lst[wave], lane);
        wh.store(hst[wave], lane);
        const uint8_t *lq = lst[wave] + r * QL::RS + 4 * g, *hq = hst[wave] + r * QH::RS + 2 * g;
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const bf16x8 ab = as_bf16x8(av[u]);
            const bf16x8 w = unpack_k6(*reinterpret_cast<const uint32_t *>(lq + 16 * u),
                                       *reinterpret_cast<const uint16_t *>(hq + 8 * u));
            const f32x4 p0 = mfma16(ab, first_half ? w : zero, f32x4{0.f, 0.f, 0.f, 0.f});
            const f32x4 p1 = mfma16(ab, first_half ? zero : w, f32x4{0.f, 0.f, 0.f, 0.f});
            const int s = u >> 3, lb = u & 7;          // super-block of the group, block within it
            // scales 2 lb and 2 lb + 1 of the super-block: bytes 2 (lb & 1) and + 1 of word lb / 2
            const uint32_t word = sc[s][lb >> 1] >> (16 * (lb & 1));
            const float s0v = dd[s] * float(int(int8_t(word & 0xFFu)));
            const float s1v = dd[s] * float(int(int8_t((word >> 8) & 0xFFu)));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc[i] = fmaf(s0v, p0[i], acc[i]);
                acc[i] = fmaf(s1v, p1[i], acc[i]);
            }
        }
    }
    uint16_t *y = static_cast<uint16_t *>(sh ? L.ys : L.y) + int64_t(it.row0) * d + c0 + r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int tok = 4 * g + i;
        if (tok < n) {
            const float w = sh ? 1.0f : L.row_weight[it.row0 + tok];
            y[int64_t(tok) * d] = f32_to_bf16(acc[i] * w);
        }
    }
}

namespace {

template <int R>
int tiles_gateup_kq_stream(int, int, int I)
{
    return I / (kqs::ROWS * R);
}

int tiles_down_kq_stream(int, int d, int)
{
    return d / (kqs::WAVES * kqs::ROWS);
}

template <int R>
hipError_t launch_gateup_kq_stream(const ExpertLaunch &L, hipStream_t s)
{
    if (L.n_tiles == 0)
        return hipSuccess;
    if (L.d % 256 != 0)
        return hipErrorInvalidValue;
    // chunk: 8, 4 or 2 blocks, dividing a quarter of d's blocks (d / 128)
    const int nq = L.d / 128;
    if (nq % 8 == 0)
        launch_k(stream_gateup_kq_kernel<8, R>, L.n_tiles, 256, 0, s, L);
    else if (nq % 4 == 0)
        launch_k(stream_gateup_kq_kernel<4, R>, L.n_tiles, 256, 0, s, L);
    else
        launch_k(stream_gateup_kq_kernel<2, R>, L.n_tiles, 256, 0, s, L);
    return hipGetLastError();
}

hipError_t launch_down_kq_stream(const ExpertLaunch &L, hipStream_t s)
{
    if (L.n_tiles == 0)
        return hipSuccess;
    if (L.I % 256 != 0 || L.d % 64 != 0)
        return hipErrorInvalidValue;
    if ((L.I / 256) % 2 == 0)
        launch_k(stream_down_kq_kernel<2>, L.n_tiles, 256, 0, s, L);
    else
        launch_k(stream_down_kq_kernel<1>, L.n_tiles, 256, 0, s, L);
    return hipGetLastError();
}

}  // namespace

// ============================================================== tile path
//
// Integer operands only.  Within a 256-element super-block the accumulators
// are in units of its d: w / d = sc q (k4, before the min) or sc (q - 32)
// (k6), exact integers of 10 and 13 bits.
//   k4: sc q <= 945 is exact in fp16, so one fp16 MFMA per 32 elements.  The
//       tokens enter as fp16 too: kq_rows_f16_kernel scales each row by a
//       power of two that puts its largest magnitude in [2^14, 2^15), where
//       every bf16 value down to 2^-31 of it keeps its 8 bits (in fp16's
//       subnormal range, which the MFMA reads as it is).  A row with a value
//       that does not is marked, and its outputs are computed from the bf16
//       row in fp32 after the tile's others (exact_rows): no token loses bits.
//   k6: sc = 16 h + l (h in -8..8, l in -8..7): 16 h (q - 32) and l (q - 32)
//       have at most 8 significant bits each, two exact bf16 MFMAs.  They carry
//       2^-15, so that the accumulators stay near the results' own magnitude
//       (d is 2^-15 of a matrix's largest weight) and reach as far.  An MFMA
//       rounds more than once on its way into its C, so two of them a block
//       straight into the accumulators lose more than the one FMA a sub-block
//       they stand for: each stage's 64 elements are summed from zero, the l
//       parts first, and then added.
// At a super-block's end the k4 accumulators take their mins off, acc -=
// (dmin / d) sum_j m_j S_j, and both move to the next unit, acc *= d / d_next;
// the result is acc d after the last (and 2^-k of the row's scale).  S_j, the
// rows' sums over the 32-element sub-blocks, comes from MFMAs against
// indicator rows (each wavefront its share of the row blocks), crosses LDS
// as 2^-5 S_j (at most 2^15) and comes back as an operand in three fp16 parts
// of 11 bits, part p times 2^11p, beside 2^-11p m_j (m_j 0..63: exact).  A
// super-block with d = 0 keeps the previous unit, scale 0.
//
// So k4 costs one MFMA per 16 x 16 x 32 block, and k6 two, with the unpacking
// (13 and 48 vector operations per fragment) shared by MB row blocks and two
// (k6: six) fp32 operations per output and super-block; applying each sub-block's
// scale and min in fp32 instead took two FMAs per output and sub-block and kept
// the vector ALU at 96 cycles a block.
//
// Error against 64 bits, as the share of values off the correctly rounded bf16
// (d 2048, I 512; this form / a sub-block at a time with the codes as 128 + q):
// act 5.4e-4 / 23e-4 on N(0, 1) tokens, 1.0e-3 / 8.6e-3 and 1.7e-3 / 5.2e-3 with
// one element of 2^10 and 2^20; y rows 7.6e-5 / 8.3e-5 (I 256: 5.8e-5 / 5.9e-5,
// 768: 8.4e-5 / 10.2e-5).  Straight into the accumulators y rows had 13.0e-5
// (I 768: 15.7e-5); summed by 32 elements 8.5e-5.  At 32768 tokens down takes
// 1795 us, by 32 elements 1848, straight 1546 (same card).
namespace kqt {
constexpr int BK = 64, ROWB = BK * 2, QROWB = BK / 2, HROWB = BK / 4;

template <bool GU_, int BM_, int TN_, int WC_, int WPC_>
struct Shape {
    static constexpr bool GU = GU_;
    static constexpr int BM = BM_, TN = TN_, WC = WC_, WPC = WPC_;   // rows, weight rows, wavefronts, workgroups per CU
    static constexpr int WAVES = WC, THREADS = 64 * WAVES;
    static constexpr int MB = BM / 16, NB = TN / WC / 16;
    static constexpr int A_BYTES = BM * ROWB, Q_BYTES = TN * QROWB, H_BYTES = GU ? 0 : TN * HROWB;
    static constexpr int STAGE = A_BYTES + Q_BYTES + H_BYTES;
    static constexpr int LA = BM / 8 / WAVES, LQ = TN / 32 / WAVES;   // copies per wavefront per stage
    static constexpr int NH = TN / 64;                                // copies of high parts per stage (k6)
    // tables of one super-block (two of each): sub-block scales (k4 [4][TN] pairs of fp16, k6 [16][TN] int8), unit ratios
    // [TN], min coefficients [TN] and mins [TN][8] fp16 (k4); then the sub-block sums [BM][4][8] fp16 (k4: three
    // parts, the fourth zero)
    static constexpr int T_SC = 16 * TN, T_R = TN * 4, T_C = GU ? TN * 4 : 0, T_M = GU ? TN * 16 : 0;
    static constexpr int TABLE = T_SC + T_R + T_C + T_M;
    static constexpr int S_BYTES = GU ? BM * 64 : 0;
    static constexpr size_t LDS = 2 * STAGE + 2 * TABLE + S_BYTES;
    static_assert(BM % (8 * WAVES) == 0 && TN % (32 * WAVES) == 0 && NH <= WAVES && TN <= THREADS && MB % WC == 0, "");
    static_assert(LDS * WPC <= 160 * 1024, "");
};
}  // namespace kqt

typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;

__device__ __forceinline__ f32x4 mfma16h(const f16x8 &a, const f16x8 &b, const f32x4 &c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// k4: 8 nibbles and a sub-block's scale (fp16, twice) -> sc q, exact fp16, in the element order 0 4 1 5 2 6 3 7 (the
// order kq_rows_f16_kernel writes the tokens in): 1024 + q (bits 0x6400 | q) or 1024 + 16 q, then one packed FMA
// that scales and takes the offset off exactly.
__device__ __forceinline__ f16x8 unpack_k4_f16(uint32_t w, uint32_t sc2)
{
    const f16x2 s = __builtin_bit_cast(f16x2, sc2);
    const f16x2 o = s * f16x2{-1024, -1024}, s16 = s * f16x2{0.0625f16, 0.0625f16}, o16 = s * f16x2{-64, -64};
    u32x4 r;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t v = w >> (8 * h);
        const f16x2 a = __builtin_bit_cast(f16x2, (v & 0x000F000Fu) | 0x64006400u);
        const f16x2 b = __builtin_bit_cast(f16x2, (v & 0x00F000F0u) | 0x64006400u);
        r[2 * h] = __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(a, s, o));
        r[2 * h + 1] = __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(b, s16, o16));
    }
    return __builtin_bit_cast(f16x8, r);
}

// k6: 8 codes and a sub-block's scale -> the two operands, times K6_SCALE
constexpr float K6_SCALE = 1.0f / 32768;
__device__ __forceinline__ void unpack_k6_pair(uint32_t lo4, uint32_t hi2, int sc, bf16x8 &hi, bf16x8 &lo)
{
    const int h16 = (sc + 8) & ~15;                // sc = 16 h + l, l in -8 .. 7
    uint32_t t = (hi2 | (hi2 << 8)) & 0x00FF00FFu;
    t = (t | (t << 4)) & 0x0F0F0F0Fu;
    const uint32_t ev = (lo4 & 0x0F0F0F0Fu) | ((t & 0x03030303u) << 4);          // elements 0, 2, 4, 6
    const uint32_t od = ((lo4 >> 4) & 0x0F0F0F0Fu) | ((t & 0x0C0C0C0Cu) << 2);   // elements 1, 3, 5, 7
    const float s1 = float(h16) * K6_SCALE, s2 = float(sc - h16) * K6_SCALE;
    const float o1 = -32.0f * s1, o2 = -32.0f * s2;
    u32x4 a, b;
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const float fe = float((ev >> (8 * h)) & 0xFFu), fo = float((od >> (8 * h)) & 0xFFu);
        // exact: at most 8 significant bits, the top half of their binary32
        a[h] = __builtin_amdgcn_perm(__float_as_uint(fmaf(fo, s1, o1)), __float_as_uint(fmaf(fe, s1, o1)), 0x07060302u);
        b[h] = __builtin_amdgcn_perm(__float_as_uint(fmaf(fo, s2, o2)), __float_as_uint(fmaf(fe, s2, o2)), 0x07060302u);
    }
    hi = __builtin_bit_cast(bf16x8, a);
    lo = __builtin_bit_cast(bf16x8, b);
}

// Gate/up: tile columns 0 .. TN/2 - 1 are gate rows nt TN/2 .., the rest the
// matching up rows; each wavefront owns all MB 16-row blocks and NB column
// blocks (gate/up: NB / 2 gate blocks and the matching up blocks, so SiLU * up
// forms in registers).  Weights are the A operand: a lane's outputs are
// columns 4g .. 4g + 3 of row r16, stored as 16-byte pieces straight to memory.
// A rows and packed codes are copied straight to LDS, one stage of 64
// elements ahead (two buffers); thread c < TN reads column c's header one
// super-block ahead and decodes it into the tables.
template <class S>
struct KqTile {
static constexpr size_t LDS = S::LDS;
static constexpr int WAVES_PER_SIMD = S::WPC * S::WAVES / 4;
static __device__ __forceinline__ void run(const ExpertLaunch &L, int block, int n_blocks, uint8_t *lds8)
{
    using namespace kqt;
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
    const int r16 = lane & 15, g = lane >> 4;

    const uint8_t *obj = sh ? L.shared_w : L.wbase + uint64_t(it.slot) * L.wstride;
    const uint32_t mbytes = k4_bytes(I, d);
    // byte offset, from the object, of tile column c's matrix and its row there
    auto col_matrix = [&](int c) -> uint32_t { return GU ? (c < TN / 2 ? 0u : mbytes) : 2 * mbytes; };
    auto col_row = [&](int c) -> uint32_t {
        return GU ? uint32_t(nt * (TN / 2) + (c < TN / 2 ? c : c - TN / 2)) : uint32_t(nt * TN + c);
    };

    // ---- stage copies (slots permuted as in the 4-bit tiles, so fragment reads are free of bank conflicts)
    [[maybe_unused]] const void *abase = GU ? L.xh
                           : static_cast<const uint8_t *>(sh ? L.act_s : L.act) + (int64_t(it.row0) + m0) * int64_t(I) * 2;
    // Offset of copy i.  Down's are worked out again for each stage (the lane index is made opaque): its products' sums
    // (below) leave no registers to keep them in.
    auto lane_of = [&]() {
        int l = lane;
        if constexpr (!GU)
            asm volatile("" : "+v"(l));
        return l;
    };
    auto a_off = [&](int i) -> uint32_t {
        const int l = lane_of(), r = 8 * (WAVES * i + wave) + (l >> 3);
        const int m = m0 + min(r, valid - 1);     // rows past the end repeat the last one and are never stored
        const uint32_t src = !GU ? uint32_t(m - m0) : sh ? uint32_t(it.row0 + m) : uint32_t(L.perm[it.row0 + m]);
        return src * uint32_t(K * 2) + uint32_t(((l & 7) ^ ((r >> 1) & 7)) << 4);
    };
    auto q_off = [&](int i) -> uint32_t {
        const int l = lane_of(), c = 32 * (WAVES * i + wave) + (l >> 1);
        return col_matrix(c) + col_row(c) * uint32_t(K / 2) + uint32_t(16 * ((l & 1) ^ ((c >> 3) & 1)));
    };
    auto h_off = [&]() -> uint32_t {
        return col_matrix(0) + uint32_t(d) * uint32_t(K / 2) + col_row(64 * (wave % S::NH) + lane_of()) * uint32_t(K / 4);
    };
    [[maybe_unused]] uint32_t aoff[S::LA], qoff[S::LQ];
    if constexpr (GU) {
#pragma unroll
        for (int i = 0; i < S::LA; ++i)
            aoff[i] = a_off(i);
#pragma unroll
        for (int i = 0; i < S::LQ; ++i)
            qoff[i] = q_off(i);
    }
    auto issue = [&](int stage, int buf) {
        uint8_t *st = lds8 + buf * STAGE;
#if defined(__HIP_DEVICE_COMPILE__)
        const __amdgpu_buffer_rsrc_t ar =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(abase), 0, 0x7fffffff, 0x00020000u);
        const __amdgpu_buffer_rsrc_t wr_ =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(obj), 0, 0x7fffffff, 0x00020000u);
#pragma unroll
        for (int i = 0; i < S::LA; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ar, (lds_void_t *)(st + (WAVES * i + wave) * 1024), 16,
                                                     GU ? aoff[i] : a_off(i), stage * ROWB, 0, 0);
#pragma unroll
        for (int i = 0; i < S::LQ; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr_, (lds_void_t *)(st + S::A_BYTES + (WAVES * i + wave) * 1024),
                                                     16, GU ? qoff[i] : q_off(i), stage * QROWB, 0, 0);
        if (!GU && wave < S::NH)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr_, (lds_void_t *)(st + S::A_BYTES + S::Q_BYTES + wave * 1024), 16,
                                                     h_off(), stage * HROWB, 0, 0);
#else
        (void)st, (void)stage;
#endif
    };

    // ---- super-block tables
    uint8_t *tables = lds8 + 2 * STAGE;
    uint16_t *sums = reinterpret_cast<uint16_t *>(lds8 + 2 * STAGE + 2 * S::TABLE);
    const int nsb = K / 256;
    u32x4 hd = {0u, 0u, 0u, 0u};                  // next super-block's header (k6: its 16 scales)
    uint16_t hd6 = 0;                             // k6: its d
    float unit = 1.0f;                            // d of the last decoded super-block
    const uint8_t *hp = nullptr;
    const uint16_t *dp = nullptr;
    if (tid < TN) {
        const uint8_t *mat = obj + col_matrix(tid);
        const uint32_t row = col_row(tid);
        if (GU) {
            hp = mat + uint32_t(I) * uint32_t(K / 2) + row * uint32_t(nsb) * 16u;
        } else {
            const K6Planes P = k6_planes(mat, uint32_t(d), uint32_t(K));
            hp = reinterpret_cast<const uint8_t *>(P.sc) + row * uint32_t(K / 16);
            dp = P.d + row * uint32_t(nsb);
        }
    }
    auto load_header = [&](int sb) {
        if (tid < TN) {
            hd = *reinterpret_cast<const u32x4 *>(hp + 16 * sb);
            if (!GU)
                hd6 = dp[sb];
        }
    };
    auto decode_header = [&](int sb) {
        if (tid >= TN)
            return;
        uint8_t *tb = tables + (sb & 1) * S::TABLE;
        const float dv = h2f(GU ? uint16_t(hd[0]) : hd6);
        const float u = dv != 0.0f ? dv : unit;
        if constexpr (GU) {
            // pairs of 6-bit values -> pairs of fp16, exact through 1024 + v
            auto pair = [](uint32_t v12) {
                const uint32_t b = (v12 & 63u) | ((v12 & 0xFC0u) << 10) | 0x64006400u;
                return __builtin_bit_cast(uint32_t, __builtin_bit_cast(f16x2, b) - f16x2{1024, 1024});
            };
            const uint32_t m3 = __builtin_amdgcn_alignbit(hd[3], hd[2], 16);   // mins 0 ..: bits 0 .. 31 of their 48
            const uint32_t v[8] = {hd[1],        hd[1] >> 12, __builtin_amdgcn_alignbit(hd[2], hd[1], 24), hd[2] >> 4,
                                   m3,           m3 >> 12,    hd[3] >> 8,                                  hd[3] >> 20};
            uint32_t p[8];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                p[j] = pair(v[j]);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                reinterpret_cast<uint32_t *>(tb)[j * TN + tid] = dv != 0.0f ? p[j] : 0u;
            *reinterpret_cast<u32x4 *>(tb + S::T_SC + S::T_R + S::T_C + tid * 16) = u32x4{p[4], p[5], p[6], p[7]};
            reinterpret_cast<float *>(tb + S::T_SC + S::T_R)[tid] = 32.0f * (h2f(uint16_t(hd[0] >> 16)) / u);
        } else {
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const uint32_t b = (hd[j >> 2] >> (8 * (j & 3))) & 0xFFu;
                tb[j * TN + tid] = dv != 0.0f ? uint8_t(b) : uint8_t(0);
            }
        }
        reinterpret_cast<float *>(tb + S::T_SC)[tid] = unit / u;
        unit = u;
    };

    auto col_of = [&](int nb) -> int {              // tile column block of this wavefront
        if (GU)
            return nb < NB / 2 ? (wave * (NB / 2) + nb) * 16 : TN / 2 + (wave * (NB / 2) + nb - NB / 2) * 16;
        return (wave * NB + nb) * 16;
    };
    f32x4 acc[NB][MB];
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int b = 0; b < MB; ++b)
            acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    // sub-block sums: this wavefront's share of its row blocks
    constexpr int SMB = GU ? MB / S::WC : 1;
    f32x4 sacc[SMB];
    auto a_frag = [&](const uint8_t *st, int r, int kb) {     // elements 8g .. 8g + 7 of block kb of row r
        return *reinterpret_cast<const u32x4 *>(st + r * ROWB + (((4 * kb + g) ^ ((r >> 1) & 7)) << 4));
    };
    auto codes = [&](const uint8_t *st, int c, int kb) {      // their codes' (low) nibbles in weight row c
        return *reinterpret_cast<const uint32_t *>(st + S::A_BYTES + c * QROWB + 16 * (kb ^ ((c >> 3) & 1)) + 4 * g);
    };
    auto compute = [&](int buf, int stage) {
        const uint8_t *st = lds8 + buf * STAGE;
        const uint8_t *sct = tables + ((stage >> 2) & 1) * S::TABLE;
        if constexpr (GU) {
#pragma unroll
            for (int kb = 0; kb < BK / 32; ++kb) {
                const int jb = (stage & 3) * 2 + kb;               // 32-element block of the super-block
                u32x4 af[MB];
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
                    af[mb] = a_frag(st, mb * 16 + r16, kb);
                const uint32_t one = r16 == jb ? 0x3C003C00u : 0u;
                const f16x8 ind = __builtin_bit_cast(f16x8, u32x4{one, one, one, one});
#pragma unroll
                for (int q = 0; q < SMB; ++q)
                    sacc[q] = mfma16h(ind, __builtin_bit_cast(f16x8, a_frag(st, (wave * SMB + q) * 16 + r16, kb)), sacc[q]);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const int c = col_of(nb) + r16;                // A fragment: weight row c
                    const uint32_t s2 = reinterpret_cast<const uint32_t *>(sct)[(stage & 3) * TN + c];
                    const f16x8 w =
                        unpack_k4_f16(codes(st, c, kb), __builtin_amdgcn_perm(s2, s2, kb ? 0x03020302u : 0x01000100u));
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb)
                        acc[nb][mb] = mfma16h(w, __builtin_bit_cast(f16x8, af[mb]), acc[nb][mb]);
                }
            }
        } else {
            // The stage's 64 elements are summed before they are added, the small parts l first.  (The second block's
            // act fragments are read again for each column block: held, they would spill.)
            constexpr int G = 4;                                   // row blocks at a time
            u32x4 af[MB];
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
                af[mb] = a_frag(st, mb * 16 + r16, 0);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                __builtin_amdgcn_sched_barrier(0);
                const int c = col_of(nb) + r16;                    // A fragment: weight row c
                bf16x8 hi[2], lo[2];
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) {
                    const uint32_t hw = *reinterpret_cast<const uint16_t *>(st + S::A_BYTES + S::Q_BYTES + c * HROWB +
                                                                            8 * kb + 2 * g);
                    const int j16 = ((stage & 3) * 2 + kb) * 2 + (g >> 1);   // 16-element sub-block
                    unpack_k6_pair(codes(st, c, kb), hw, int(int8_t(sct[j16 * TN + c])), hi[kb], lo[kb]);
                }
#pragma unroll
                for (int m0_ = 0; m0_ < MB; m0_ += G) {
                    f32x4 part[G];
                    u32x4 a1[G];
#pragma unroll
                    for (int q = 0; q < G; ++q) {
                        part[q] = mfma16(lo[0], as_bf16x8(af[m0_ + q]), f32x4{0.f, 0.f, 0.f, 0.f});
                        a1[q] = a_frag(st, (m0_ + q) * 16 + r16, 1);
                    }
#pragma unroll
                    for (int q = 0; q < G; ++q)
                        part[q] = mfma16(lo[1], as_bf16x8(a1[q]), part[q]);
#pragma unroll
                    for (int q = 0; q < G; ++q)
                        part[q] = mfma16(hi[0], as_bf16x8(af[m0_ + q]), part[q]);
#pragma unroll
                    for (int q = 0; q < G; ++q)
                        part[q] = mfma16(hi[1], as_bf16x8(a1[q]), part[q]);
#pragma unroll
                    for (int q = 0; q < G; ++q)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            acc[nb][m0_ + q][i] += part[q][i];
                }
            }
        }
    };
    auto clear_sums = [&]() {
#pragma unroll
        for (int q = 0; q < SMB; ++q)
            sacc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    // a lane holds sub-blocks 4g .. 4g + 3 (g < 2) of row r16: their three fp16 parts, in the operand's layout
    // (part p times 2^11p, against mins times 2^-11p: each part keeps its 11 bits)
    auto store_sums = [&]() {
        if constexpr (GU) {
            if (g < 2) {
#pragma unroll
                for (int q = 0; q < SMB; ++q) {
                    uint16_t *sp = sums + ((wave * SMB + q) * 16 + r16) * 32 + 4 * g;
                    f32x4 s = sacc[q] * 0.03125f;
#pragma unroll
                    for (int p = 0; p < 3; ++p) {
                        uint16_t h[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            h[i] = f16_bits(s[i]);
                            s[i] = (s[i] - h2f(h[i])) * 2048.0f;
                        }
                        *reinterpret_cast<uint2 *>(sp + 8 * p) =
                            make_uint2(uint32_t(h[0]) | (uint32_t(h[1]) << 16), uint32_t(h[2]) | (uint32_t(h[3]) << 16));
                    }
                }
            }
        }
    };
    // super-block sb - 1 ends: its mins come off, and the accumulators move to super-block sb's unit
    const _Float16 ps = g == 0 ? _Float16(1.0f) : g == 1 ? _Float16(0x1p-11f) : _Float16(0x1p-22f);   // (part 3 is 0)
    [[maybe_unused]] const f16x8 part_scale = {ps, ps, ps, ps, ps, ps, ps, ps};
    auto finish = [&](int sb) {
        const uint8_t *tb = tables + (sb & 1) * S::TABLE, *to = tables + ((sb & 1) ^ 1) * S::TABLE;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const f32x4 r = *reinterpret_cast<const f32x4 *>(tb + S::T_SC + (col_of(nb) + 4 * g) * 4);
            if constexpr (GU) {
                const f16x8 mf =
                    *reinterpret_cast<const f16x8 *>(to + S::T_SC + S::T_R + S::T_C + (col_of(nb) + r16) * 16) * part_scale;
                f32x4 cm = *reinterpret_cast<const f32x4 *>(to + S::T_SC + S::T_R + (col_of(nb) + 4 * g) * 4);
                cm = cm * r;
#pragma unroll
                for (int m0_ = 0; m0_ < MB; m0_ += 2) {
                    __builtin_amdgcn_sched_barrier(0);   // (two row blocks at a time: hoisted reads would spill)
                    f32x4 m[2];
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const f16x8 pa = *reinterpret_cast<const f16x8 *>(
                            sums + ((m0_ + q) * 16 + r16) * 32 + 8 * g);
                        m[q] = mfma16h(mf, pa, f32x4{0.f, 0.f, 0.f, 0.f});
                    }
#pragma unroll
                    for (int q = 0; q < 2; ++q)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            acc[nb][m0_ + q][i] = fmaf(-cm[i], m[q][i], acc[nb][m0_ + q][i] * r[i]);
                }
            } else {
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        acc[nb][mb][i] *= r[i];
            }
        }
    };

    // token of tile row `row`
    auto token_of = [&](int row) -> int { return sh ? it.row0 + m0 + row : L.perm[it.row0 + m0 + row]; };
    // Outputs of the tile's marked rows from their bf16 tokens, sub-block by sub-block in fp32 as on the stream path
    // (the products plain FMAs): two threads per column, in either tile form, take alternate super-blocks.  A row adds
    // 24 us to its tiles at d 2048 (vector operations of two threads' serial sums); an N(0, 1) token has a value under
    // 2^-31 of its largest about three times in a million.
    auto exact_rows = [&](const uint64_t (&marks)[BM / 64]) {
        if constexpr (GU) {
            constexpr int NC = TN / 2;
            static_assert(2 * NC <= S::THREADS, "");
            const int c = min(tid >> 1, NC - 1), part = tid & 1;
            const uint8_t *q0 = obj + (nt * NC + c) * (d / 2), *h0 = obj + I * (d / 2) + (nt * NC + c) * nsb * 16;
#pragma unroll
            for (int b = 0; b < BM; b += 64) {
                for (uint64_t m64 = marks[b / 64]; m64; m64 &= m64 - 1) {     // (the same for every wavefront)
                    const int row = b + __builtin_ctzll(m64);
                    const uint32_t *x = reinterpret_cast<const uint32_t *>(static_cast<const uint16_t *>(L.x) +
                                                                           int64_t(token_of(row)) * d);
                    float v[2] = {0.f, 0.f};
#pragma unroll 1
                    for (int sb = part; sb < nsb; sb += 2) {
                        const u32x4 hdr[2] = {*reinterpret_cast<const u32x4 *>(h0 + sb * 16),
                                              *reinterpret_cast<const u32x4 *>(h0 + mbytes + sb * 16)};
#pragma unroll 4
                        for (int j = 0; j < 8; ++j)
#pragma unroll
                            for (int m = 0; m < 2; ++m) {
                                const u32x4 w = *reinterpret_cast<const u32x4 *>(q0 + m * mbytes + 128 * sb + 16 * j);
                                float a, o, p = 0.f, sum = 0.f;
                                k4_coef(hdr[m], j, a, o);
#pragma unroll
                                for (int e = 0; e < 32; e += 2) {
                                    const uint32_t xx = x[128 * sb + 16 * j + e / 2];
                                    const float x0 = __uint_as_float(xx << 16), x1 = __uint_as_float(xx & 0xFFFF0000u);
                                    p = fmaf(x0, float((w[e >> 3] >> (4 * (e & 7))) & 15u), p);
                                    p = fmaf(x1, float((w[e >> 3] >> (4 * (e & 7) + 4)) & 15u), p);
                                    sum += x0;
                                    sum += x1;
                                }
                                v[m] = fmaf(a, p, v[m]);
                                v[m] = fmaf(-o, sum, v[m]);
                            }
                    }
                    v[0] += __shfl_xor(v[0], 1);
                    v[1] += __shfl_xor(v[1], 1);
                    if (part == 0 && tid < 2 * NC)
                        static_cast<uint16_t *>(sh ? L.act_s : L.act)[(int64_t(it.row0) + m0 + row) * I + nt * NC + c] =
                            f32_to_bf16(silu(v[0]) * v[1]);
                }
            }
        }
    };

    const int nk = K / BK;
    if (GU)
        for (int r = tid; r < BM; r += S::THREADS)
            *reinterpret_cast<u32x4 *>(sums + r * 32 + 24) = u32x4{0u, 0u, 0u, 0u};
    load_header(0);
    issue(0, 0);
    decode_header(0);
    for (int sb = 0; sb < nsb; ++sb) {
        if (sb + 1 < nsb)
            load_header(sb + 1);
        clear_sums();
#pragma unroll 1
        for (int q = 0; q < 4; ++q) {
            const int kt = 4 * sb + q;
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(0x0070);     // vmcnt(0) lgkmcnt(0): this stage and the tables are in LDS
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (kt + 1 < nk)
                issue(kt + 1, (kt + 1) & 1);
            compute(kt & 1, kt);
        }
        store_sums();
        if (sb + 1 < nsb)
            decode_header(sb + 1);
        else if (tid < TN)                          // after the last, the unit is 1
            reinterpret_cast<float *>(tables + (nsb & 1) * S::TABLE + S::T_SC)[tid] = GU ? unit : unit / K6_SCALE;
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);         // lgkmcnt(0): the sums and the tables (stage copies stay in flight)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        finish(sb + 1);
    }
    if (!slot_gen_ok(it, gnow, L.status))
        return;

    // ---- epilogue: lane holds columns 4g .. 4g + 3 of each block of row r16; two blocks at a time are regrouped
    // so that each lane stores 16 contiguous bytes
    const int64_t rowbase = int64_t(it.row0) + m0;
    uint64_t marks[BM / 64] = {};
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        const int row = mb * 16 + r16;
        bool in = row < valid;
        constexpr int OB = GU ? NB / 2 : NB;        // output blocks
        uint32_t lo[OB], hi[OB];
        if constexpr (GU) {
            const int xe = in ? int(L.xexp[token_of(row)]) : 0, k = -xe;
            in = in && xe != KQ_INEXACT;            // (exact_rows stores those; lanes 16 apart hold the same row)
            marks[mb / 4] |= (__ballot(xe == KQ_INEXACT) & 0xFFFFull) << (16 * (mb % 4));
#pragma unroll
            for (int nb = 0; nb < OB; ++nb) {
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    v[i] = silu(ldexpf(acc[nb][mb][i], k)) * ldexpf(acc[nb + OB][mb][i], k);
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
        dst += wave * OB * 16;
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
    exact_rows(marks);
}
};

template <class S>
__global__ void __launch_bounds__(S::THREADS, S::WPC *S::WAVES / 4) tile_kq_kernel(ExpertLaunch L)
{
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds8[];
    KqTile<S>::run(L, int(blockIdx.x), int(gridDim.x), lds8);
}

// Tokens for the k4 tiles: xh[t] = fp16(2^k x[t]) with elements 0 4 1 5 2 6 3 7 of each group of eight, k = xexp[t]
// putting the row's largest magnitude in [2^14, 2^15) (0 for rows of zeros or with an infinity or NaN, whose
// outputs are not numbers either way; at most 127).  A row with an element that fp16 does not hold exactly gets
// xexp[t] = KQ_INEXACT.  One wavefront per row; the row is read twice, the second time from the caches.
__global__ void __launch_bounds__(256) kq_rows_f16_kernel(const uint16_t *__restrict__ x, uint16_t *__restrict__ xh,
                                                          int8_t *__restrict__ xexp, int T, int d,
                                                          const DevCount *__restrict__ tiles)
{
    if (tiles && tiles->n_items == 0)
        return;                                   // no tile reads the copy
    const int t = int(blockIdx.x) * 4 + int(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (t >= T)
        return;
    const u32x4 *src = reinterpret_cast<const u32x4 *>(x + int64_t(t) * d);
    u32x4 *dst = reinterpret_cast<u32x4 *>(xh + int64_t(t) * d);
    uint32_t m = 0;
    for (int c = lane; c < d / 8; c += 64) {
        const u32x4 v = src[c];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            m = max(m, max(v[i] & 0x7FFFu, (v[i] >> 16) & 0x7FFFu));
    }
    // (magnitudes of bf16 bits order as integers; up to 0x7FFF they are exact as floats)
    m = uint32_t(wave_max(float(m)));
    const int e = max(int(m >> 7), 1);
    const int k = (m == 0u || e == 255) ? 0 : min(141 - e, 127);
    bool exact = true;
    for (int c = lane; c < d / 8; c += 64) {
        const u32x4 v = src[c];
        uint16_t h[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float f = ldexpf(__uint_as_float((i & 1) ? v[i / 2] & 0xFFFF0000u : v[i / 2] << 16), k);
            h[i] = f16_bits(f);
            exact = exact && h2f(h[i]) == f;
        }
        dst[c] = u32x4{uint32_t(h[0]) | (uint32_t(h[4]) << 16), uint32_t(h[1]) | (uint32_t(h[5]) << 16),
                       uint32_t(h[2]) | (uint32_t(h[6]) << 16), uint32_t(h[3]) | (uint32_t(h[7]) << 16)};
    }
    const bool all = __all(exact) || e == 255;
    if (lane == 0)
        xexp[t] = all ? int8_t(k) : KQ_INEXACT;
}

hipError_t launch_kq_rows_f16(const void *x, void *xh, int8_t *xexp, int T, int d, const DevCount *tiles, hipStream_t s)
{
    if (T == 0)
        return hipSuccess;
    launch_k(kq_rows_f16_kernel, unsigned((T + 3) / 4), 256, 0, s, static_cast<const uint16_t *>(x),
             static_cast<uint16_t *>(xh), xexp, T, d, tiles);
    return hipGetLastError();
}

namespace {

template <class S>
int kq_tiles(int nrows, int d, int I)
{
    return (nrows + S::BM - 1) / S::BM * (S::GU ? I / (S::TN / 2) : d / S::TN);
}

template <class S>
TileGeom kq_geom(int d, int I)
{
    return TileGeom{S::BM, S::GU ? I / (S::TN / 2) : d / S::TN};
}

template <class S>
hipError_t launch_kq_tile(const ExpertLaunch &L, hipStream_t s)
{
    if (L.n_tiles == 0)
        return hipSuccess;
    if (L.d % 256 != 0 || L.I % 256 != 0)
        return hipErrorInvalidValue;
    launch_k(tile_kq_kernel<S>, L.n_tiles, S::THREADS, S::LDS, s, L);
    return hipGetLastError();
}

template <bool GU>
using KqSmall = kqt::Shape<GU, 64, 128, 4, 3>;
template <bool GU>
using KqBig = kqt::Shape<GU, 128, 256, 4, 2>;

// The 64-row gate/up tiles and the stream list in one launch (both_kernel).
// Measured (MI355X, E 512, d 2048, I 512, K 10, router bias 0.3 ln Zipf(1.5);
// us): two launches 28 + 83 (128 tokens), 36 + 101 (251), 95 + 121 (1013);
// together 92, 124, 207.  Down stays in two: its stream kernel runs five
// workgroups per CU alone (96 registers), three in a joint kernel (137, both
// lists' live together; LDS would leave four): 130 against 21 + 88 with tiles
// that did not sum by stage (24 now).
hipError_t launch_gateup_kq_both(const ExpertLaunch &T, const ExpertLaunch &S, hipStream_t s)
{
    using Tile = KqTile<KqSmall<true>>;
    const int nq = S.d / 128;
    if (nq % 8 == 0)
        return launch_both<Tile, KqStreamGateUp<8, 2>>(T, S, s);
    if (nq % 4 == 0)
        return launch_both<Tile, KqStreamGateUp<4, 2>>(T, S, s);
    return launch_both<Tile, KqStreamGateUp<2, 2>>(T, S, s);
}

template <template <bool> class S, int R>
const KernelSet kq_set{kq_tiles<S<true>>, tiles_gateup_kq_stream<R>, kq_tiles<S<false>>, tiles_down_kq_stream,
                       kq_geom<S<true>>, kq_geom<S<false>>,
                       launch_kq_tile<S<true>>, launch_gateup_kq_stream<R>,
                       launch_kq_tile<S<false>>, launch_down_kq_stream,
                       R == 2 && S<true>::BM == 64 ? launch_gateup_kq_both : nullptr};

}  // namespace

// The tile form by the mean rows per expert; the two are bit-identical (the
// same chain of operations per output), so the choice is the launch's.
// Measured (MI355X, E 512, d 2048, I 512, K 10; gate/up + down, us):
//   mean rows   64 x 128   128 x 256   (per-sub-block scaling, 128 x 128)
//      20       190+169    316+245        526+413
//      59       318+285    393+327           -
//      80       462+407    393+338        732+642
//     640      2559+2162  1998+1737      4134+3573
const KernelSet &kq_kernels(uint64_t rows, uint64_t E, uint64_t items)
{
    // (R of the stream gate/up by the launch's items, as for the 4-bit kernels: E 128, K 4, 16 tokens, 48 slots 166 us a
    // step, 171 with R = 2; router bias 0.3 ln Zipf(1.5), R = 1,
    // R = 2, us: T 1 9.7, 11.4; T 4 14.2, 15.4; T 16 32.6, 30.6; T 128 93, 85; T 251 114, 103; T 1013 132, 124)
    if (items < 32 && rows <= 64 * E)
        return kq_set<KqSmall, 1>;
    return rows <= 64 * E ? kq_set<KqSmall, 2> : kq_set<KqBig, 2>;
}

hipError_t init_kq_attributes()
{
    for (const void *k : {reinterpret_cast<const void *>(&tile_kq_kernel<KqSmall<true>>),
                          reinterpret_cast<const void *>(&tile_kq_kernel<KqSmall<false>>),
                          reinterpret_cast<const void *>(&tile_kq_kernel<KqBig<true>>),
                          reinterpret_cast<const void *>(&tile_kq_kernel<KqBig<false>>)}) {
        const hipError_t e = allow_large_lds(k);
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

}  // namespace msi
