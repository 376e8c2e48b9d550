// dot_f32.h -- 16 x 16 tiles of fp32 dot products (fp32 layers: router logits,
// gate/up and down), gfx950.
//
// One thread per output, one FMA per element in ascending k, so a result
// does not depend on the tiling.  The rows of both operands are read as whole
// 16-byte pieces along k and shared through LDS, one chunk of 128 elements in
// registers ahead; rows are padded by 16 bytes, which puts the 16 columns' LDS
// reads on distinct banks.  The chain of dependent FMAs (d of them) is then
// what a tile takes; reading both operands element by element from memory
// took a memory round trip per element (d 256, I 128, 64 tokens, 16 experts:
// gate/up 60 us, down 28 us).
#pragma once

#include "common.h"

namespace msi {
namespace f32t {

constexpr int ROWS = 16, COLS = 16, KC = 128, LD = KC + 4, PIECES = KC / 4;

// NM weight matrices against one set of rows
template <int NM>
struct Stage {
    f32x4 v[1 + NM][16][LD / 4];
};

// acc[m] = row(threadIdx / 16) . (w[m] + wrow(threadIdx % 16) * K), K a multiple of KC.  row(q) is the address of
// row q of the tile and wrow(c) the matrix row of tile column c; 256 threads, all of them.
template <int NM, typename Row, typename WRow>
__device__ __forceinline__ void dot(Stage<NM> &lds, Row row, const float *const (&w)[NM], WRow wrow, int K,
                                    float (&acc)[NM])
{
    const int tid = threadIdx.x, r = tid / COLS, c = tid % COLS;
    const int lr = tid / PIECES, lp = tid % PIECES;      // this thread copies rows lr, lr + 8 of every operand
    const float *src[1 + NM][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        src[0][h] = row(lr + 8 * h);
#pragma unroll
        for (int m = 0; m < NM; ++m)
            src[1 + m][h] = w[m] + int64_t(wrow(lr + 8 * h)) * K;
    }
    f32x4 v[1 + NM][2];
    auto load = [&](int k0) {
#pragma unroll
        for (int m = 0; m < 1 + NM; ++m)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                v[m][h] = *reinterpret_cast<const f32x4 *>(src[m][h] + k0 + 4 * lp);
    };
#pragma unroll
    for (int m = 0; m < NM; ++m)
        acc[m] = 0.f;
    load(0);
    for (int k0 = 0; k0 < K; k0 += KC) {
        __syncthreads();                                 // the last chunk's reads are done
#pragma unroll
        for (int m = 0; m < 1 + NM; ++m)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                lds.v[m][lr + 8 * h][lp] = v[m][h];
        __syncthreads();
        if (k0 + KC < K)
            load(k0 + KC);
#pragma unroll 8
        for (int p = 0; p < PIECES; ++p) {
            const f32x4 a = lds.v[0][r][p];
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                const f32x4 b = lds.v[1 + m][c][p];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    acc[m] = fmaf(a[i], b[i], acc[m]);
            }
        }
    }
}

}  // namespace f32t
}  // namespace msi
