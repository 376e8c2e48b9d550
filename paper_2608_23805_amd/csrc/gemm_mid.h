// gemm_mid.h -- tiles of 32, 64 and 128 rows for the tile path and the router
// logits (gemm_ring.h holds the 256-row form), gfx950: launches in which few
// rows meet each weight row, bound by streaming the weights or, for the
// router and the shared expert of a small batch, by how many CUs they reach.
//
// A workgroup owns BM rows x TN weight rows (gate/up: TN / 2 gate and the
// TN / 2 matching up rows, so SiLU(gate) * up forms in registers); its WR x WC
// wavefronts split them into blocks of v_mfma_f32_16x16x32_bf16 with the
// weights as the A operand.  K advances in stages of 64 elements: whole
// 128-byte lines of the BM + TN rows are copied straight into one of NBUF LDS
// stage buffers, NBUF - 1 stages in flight while one is multiplied.  Where
// LDS allows, two workgroups share a CU, so that one's first loads and
// epilogue run beside the other's stream.
//
// Every output element is the same chain of MFMAs over ascending K as in the
// 256-row form, with the same epilogue arithmetic, so the results are
// bit-identical and a launch may take any form.
#pragma once

#include "common.h"
#include "gemm_ring.h"
#include "kernels.h"

namespace msi {

// Shape of one instantiation: BM rows x TN weight rows, WR x WC wavefronts,
// NBUF stage buffers, WPC workgroups per CU.
template <int BM_, int TN_, int WR_, int WC_, int NBUF_, int WPC_>
struct MidShape {
    static constexpr int BM = BM_, TN = TN_, WR = WR_, WC = WC_, NBUF = NBUF_, WPC = WPC_;
    static constexpr int WAVES = WR * WC, THREADS = 64 * WAVES;
    static constexpr int BK = 64, ROWB = BK * 2;             // K elements per stage, bytes per stage row
    static constexpr int STAGE = (BM + TN) * ROWB;
    static constexpr int MB = BM / WR / 16, NB = TN / WC / 16;   // 16x16 blocks per wavefront
    static constexpr int LA = BM / 8 / WAVES;                // A copy instructions (8 rows each) per wavefront per stage
    static constexpr int LB = TN / 8 / WAVES;                // B copy instructions
    static constexpr int LPS = LA + LB;
    static constexpr size_t LDS = size_t(NBUF) * STAGE;
    static_assert(BM % (8 * WAVES) == 0 && TN % (8 * WAVES) == 0 && BM % (16 * WR) == 0 && TN % (16 * WC) == 0, "");
    static_assert(LDS * WPC <= 160 * 1024 && LPS * (NBUF - 2) < 64, "");
};

// The 64-row shape, alone and beside the stream list (less LDS there, so that three workgroups share a CU as the
// stream kernels' do).
using Mid64 = MidShape<64, 128, 1, 4, 3, 2>;
using Mid64Both = MidShape<64, 128, 1, 4, 2, 3>;

template <RingMode MODE, class S>
struct MidTile {
static constexpr size_t LDS = S::LDS;
static constexpr int WAVES_PER_SIMD = S::WPC * S::WAVES / 4;
static __device__ __forceinline__ void run(const ExpertLaunch &L, int block, int n_blocks, uint8_t *lds8)
{
    constexpr int BM = S::BM, TN = S::TN, NBUF = S::NBUF, WAVES = S::WAVES, BK = S::BK, ROWB = S::ROWB,
                  STAGE = S::STAGE, MB = S::MB, NB = S::NB, LA = S::LA, LB = S::LB, LPS = S::LPS;
    constexpr bool GU = MODE == RingMode::GateUp;
    constexpr bool RT = MODE == RingMode::Router;

    int n_items = 1, n_tiles = 0;
    const int t = RT ? xcd_swizzle(block, n_blocks) : launch_tile(L, block, n_blocks, n_items, n_tiles);
    if (t < 0)
        return;                                   // past the device-built list's tiles
    const WorkItem it = RT ? WorkItem{-1, -1, 0u, 0, L.T, 0} : L.items[find_item(L.items, n_items, t)];
    // the generation word is read here and compared before the stores: no wait between the item and the copies
    const uint32_t gnow = RT ? 0u : slot_gen_now(it, L.gen_dev);
    const int d = L.d, I = L.I;
    const int K = (GU || RT) ? d : I;
    const int ntn = RT ? (L.E + TN - 1) / TN : GU ? I / (TN / 2) : d / TN;
    const int local = t - it.tile0;
    const int m0 = (local / ntn) * BM;
    const int nt = local % ntn;
    const int valid = min(BM, it.nrows - m0);
    const bool sh = it.slot < 0;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);   // (uniform: copy destinations)

    // ---- copy addressing: instruction i of this wavefront covers the 8 stage rows from 8 (WAVES i + wave) on,
    // lane l row l / 8, slot l % 8; slot s of row r holds 16-byte chunk s ^ ((r / 2) % 8), which puts the 16
    // rows of a fragment read on distinct banks
    const int rl = lane >> 3, sl = lane & 7;
    const void *abase = (GU || RT) ? L.x
                                   : static_cast<const uint8_t *>(sh ? L.act_s : L.act) +
                                         (int64_t(it.row0) + m0) * int64_t(I) * 2;
    uint32_t aoff[LA];
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int r = 8 * (WAVES * i + wave) + rl;
        const int m = m0 + min(r, valid - 1);     // rows past the end repeat the last one and are never stored
        const uint32_t src = !(GU || RT) ? uint32_t(m - m0) : !sh && GU ? uint32_t(L.perm[it.row0 + m])
                                                                         : uint32_t(it.row0 + m);
        aoff[i] = src * uint32_t(K * 2) + uint32_t((sl ^ ((r >> 1) & 7)) << 4);
    }
    const uint8_t *wobj = RT ? L.wbase : sh ? L.shared_w : L.wbase + uint64_t(it.slot) * L.wstride;
    const uint8_t *bbase = (GU || RT) ? wobj : wobj + uint64_t(2) * I * d * 2;   // Wd follows Wg, Wu
    uint32_t boff[LB];
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        const int r = 8 * (WAVES * i + wave) + rl;
        int src = GU ? (r < TN / 2 ? nt * (TN / 2) + r : I + nt * (TN / 2) + (r - TN / 2)) : nt * TN + r;
        if (RT && src >= L.E)
            src = L.E - 1;                        // (never stored)
        boff[i] = uint32_t(src) * uint32_t(K * 2) + uint32_t((sl ^ ((r >> 1) & 7)) << 4);
    }
    const __amdgpu_buffer_rsrc_t ar =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(abase), 0, 0x7fffffff, ring::RSRC_FLAGS);
    const __amdgpu_buffer_rsrc_t br =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(bbase), 0, 0x7fffffff, ring::RSRC_FLAGS);
    const int nstage = K / BK;                    // >= 2 (K is a multiple of 128)
    auto issue = [&](int stage, int buf) {
        uint8_t *b = lds8 + buf * STAGE;
#pragma unroll
        for (int i = 0; i < LB; ++i)
            dma16_lds(br, b + BM * ROWB + (WAVES * i + wave) * 1024, boff[i], stage * ROWB);
#pragma unroll
        for (int i = 0; i < LA; ++i)
            dma16_lds(ar, b + (WAVES * i + wave) * 1024, aoff[i], stage * ROWB);
    };

    const int r16 = lane & 15, g = lane >> 4;
    const int wm = wave / S::WC, wn = wave % S::WC;
    // first stage row of weight block a (gate/up: the wavefront's gate blocks, then the matching up blocks)
    auto wrow = [&](int a) {
        if (GU)
            return a < NB / 2 ? (wn * (NB / 2) + a) * 16 : TN / 2 + (wn * (NB / 2) + a - NB / 2) * 16;
        return (wn * NB + a) * 16;
    };
    f32x4 acc[NB][MB];   // [weight block][row block]
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int q = 0; q < MB; ++q)
            acc[a][q] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto compute = [&](int buf) {
        const uint8_t *b = lds8 + buf * STAGE;
#pragma unroll
        for (int kb = 0; kb < BK / 32; ++kb) {
            const uint32_t fo = uint32_t(r16 * ROWB + (((4 * kb + g) ^ ((r16 >> 1) & 7)) << 4));
            u32x4 fw[NB], fx[MB];
#pragma unroll
            for (int a = 0; a < NB; ++a)
                fw[a] = *reinterpret_cast<const u32x4 *>(b + BM * ROWB + wrow(a) * ROWB + fo);
#pragma unroll
            for (int q = 0; q < MB; ++q)
                fx[q] = *reinterpret_cast<const u32x4 *>(b + ((wm * MB + q) * 16) * ROWB + fo);
#pragma unroll
            for (int q = 0; q < MB; ++q)
#pragma unroll
                for (int a = 0; a < NB; ++a)
                    acc[a][q] = mfma16(as_bf16x8(fw[a]), as_bf16x8(fx[q]), acc[a][q]);
        }
    };

    constexpr int AHEAD = NBUF - 1;               // stages in flight beside the one multiplied
#pragma unroll
    for (int j = 0; j < AHEAD; ++j)
        if (j < nstage)
            issue(j, j);
    int cur = 0, nxt = AHEAD;
    for (int s = 0; s < nstage; ++s) {
        // stage s has landed; the buffer of stage s + AHEAD was last read at s - 1
        if (s + AHEAD <= nstage)
            __builtin_amdgcn_s_waitcnt(VMCNT_WAIT(LPS * (AHEAD - 1)));
        else
            __builtin_amdgcn_s_waitcnt(VMCNT_WAIT(0));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (s + AHEAD < nstage)
            issue(s + AHEAD, nxt);
        compute(cur);
        cur = cur == NBUF - 1 ? 0 : cur + 1;
        nxt = nxt == NBUF - 1 ? 0 : nxt + 1;
    }
    if (!RT && !slot_gen_ok(it, gnow, L.status))
        return;

    // ---- epilogue: lane holds row 16 q + r16 of the wavefront's rows and features 4 g .. 4 g + 3 of each block
    const int64_t rowbase = int64_t(it.row0) + m0;
    if constexpr (GU) {
        uint16_t *base = static_cast<uint16_t *>(sh ? L.act_s : L.act) + rowbase * I + nt * (TN / 2) + wn * (NB / 2) * 16;
#pragma unroll
        for (int q = 0; q < MB; ++q) {
            const int row = (wm * MB + q) * 16 + r16;
            uint32_t lo[NB / 2], hi[NB / 2];
#pragma unroll
            for (int a = 0; a < NB / 2; ++a) {
                lo[a] = pack_bf16x2_hw(silu_hw(acc[a][q][0]) * acc[a + NB / 2][q][0],
                                       silu_hw(acc[a][q][1]) * acc[a + NB / 2][q][1]);
                hi[a] = pack_bf16x2_hw(silu_hw(acc[a][q][2]) * acc[a + NB / 2][q][2],
                                       silu_hw(acc[a][q][3]) * acc[a + NB / 2][q][3]);
            }
            if constexpr (NB == 2) {
                if (row < valid)
                    *reinterpret_cast<uint2 *>(base + int64_t(row) * I + 4 * g) = make_uint2(lo[0], hi[0]);
            } else {
#pragma unroll
                for (int k = 0; k < NB / 4; ++k) {
                    const uint4 v = gather16(lo[2 * k], hi[2 * k], lo[2 * k + 1], hi[2 * k + 1]);
                    if (row < valid)
                        *reinterpret_cast<uint4 *>(base + int64_t(row) * I + 32 * k + 8 * g) = v;
                }
            }
        }
    } else if constexpr (RT) {
        const int E = L.E;
#pragma unroll
        for (int q = 0; q < MB; ++q) {
            const int row = (wm * MB + q) * 16 + r16;
            if (row < valid) {
#pragma unroll
                for (int a = 0; a < NB; ++a) {
                    const int c = nt * TN + wrow(a) + 4 * g;
                    float *dst = L.logits + (rowbase + row) * E + c;
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (c + j < E)
                            dst[j] = acc[a][q][j] + (L.bias ? L.bias[c + j] : 0.0f);
                }
            }
        }
    } else {
        uint16_t *base = static_cast<uint16_t *>(sh ? L.ys : L.y) + rowbase * d + nt * TN + wn * NB * 16;
        const float *rw = (sh || !L.row_weight) ? nullptr : L.row_weight + rowbase;
        float wq[MB];
#pragma unroll
        for (int q = 0; q < MB; ++q) {
            const int row = (wm * MB + q) * 16 + r16;
            wq[q] = (rw && row < valid) ? rw[row] : 1.0f;
        }
#pragma unroll
        for (int q = 0; q < MB; ++q) {
            const int row = (wm * MB + q) * 16 + r16;
            uint32_t lo[NB], hi[NB];
#pragma unroll
            for (int a = 0; a < NB; ++a) {
                lo[a] = pack_bf16x2_hw(acc[a][q][0] * wq[q], acc[a][q][1] * wq[q]);
                hi[a] = pack_bf16x2_hw(acc[a][q][2] * wq[q], acc[a][q][3] * wq[q]);
            }
#pragma unroll
            for (int k = 0; k < NB / 2; ++k) {
                const uint4 v = gather16(lo[2 * k], hi[2 * k], lo[2 * k + 1], hi[2 * k + 1]);
                if (row < valid)
                    *reinterpret_cast<uint4 *>(base + int64_t(row) * d + 32 * k + 8 * g) = v;
            }
        }
    }
}
};

template <RingMode MODE, class S>
__global__ void __launch_bounds__(S::THREADS, S::WPC * S::WAVES / 4) mid_gemm_kernel(ExpertLaunch L)
{
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds8[];
    MidTile<MODE, S>::run(L, int(blockIdx.x), int(gridDim.x), lds8);
}

}  // namespace msi
