// Address arithmetic of linear_split_kernel, called by the kernel and by the
// host-side bounds checker (a CPU build of the library used by the tests).
#pragma once

#include <stdint.h>

#include "common.hpp"

namespace cliff {

struct LinSplitArgs {
    const float* x;
    const float* w;
    const float* bias;
    float* y;
    int64_t B;
    int64_t n_tile;  // tiles of 32 rows of X
    int C_in, C_out;
    SignMasks sign;
    ActParams act;
};

// NB blades; N = 32 RT output columns, K = 16 KQ input columns.
struct LinSplitShape {
    int NB, RT, KQ;
    __host__ __device__ constexpr int N() const { return 32 * RT; }
    __host__ __device__ constexpr int K() const { return 16 * KQ; }
    // LDS bytes: one part of the expanded weight, [chunk of 8 K][N] of 16
    // bytes; all three; with the bias, gate coefficients and gate biases
    __host__ __device__ constexpr int plane() const { return 2 * KQ * N() * 16; }
    __host__ __device__ constexpr int tail() const { return 3 * plane(); }
    __host__ __device__ constexpr int lds_bytes() const { return tail() + (2 * N() + N() / NB) * 4; }
    __host__ __device__ constexpr int items() const { return 2 * KQ * (N() / NB); }
};

// Weight item e: chunk e / C_out of 8 K slots for output channel e % C_out;
// K slot u of it is blade (8 chunk + u) % NB of input channel (8 chunk + u) / NB.
__host__ __device__ inline int lsp_w_co(const LinSplitShape& S, int e) { return e % (S.N() / S.NB); }
__host__ __device__ inline int lsp_w_chunk(const LinSplitShape& S, int e) { return e / (S.N() / S.NB); }
__host__ __device__ inline int lsp_w_float(const LinSplitShape& S, int ci, int co)
{
    return (ci * (S.N() / S.NB) + co) * S.NB;
}
// LDS byte of (chunk, output column n) in a plane
__host__ __device__ inline int lsp_a_byte(const LinSplitShape& S, int chunk, int n)
{
    return (chunk * S.N() + n) * 16;
}

// A load instruction takes 64 contiguous bytes of 16 rows (whole requests;
// 32 rows by 32 bytes ask for every one twice): load h of K group s reads the
// 4 floats 4 (lane / 16) ... of row 16 h + lane % 16.  Lane rows 1 and 3 of
// load 0 then change places with lane rows 0 and 2 of load 1 (16 lanes each),
// after which every lane holds the 8 values of slots 8 (lane / 32) ... of row
// lane % 32.
__host__ __device__ constexpr int lsp_x_float(const LinSplitShape& S, int lane, int s, int h)
{
    return (16 * h + (lane & 15)) * S.K() + 16 * s + 4 * (lane >> 4);
}
// Rows of tile t inside the batch.
__host__ __device__ inline int lsp_rows(const LinSplitArgs& a, int64_t t)
{
    const int64_t left = a.B - 32 * t;
    return (int)(left < 32 ? left : 32);
}
// Output column of accumulator registers 4 q ... 4 q + 3 of row tile rt
// (the lane's row is lane % 32).
__host__ __device__ inline int lsp_y_col(const LinSplitShape&, int lane, int rt, int q)
{
    return 32 * rt + 8 * q + 4 * (lane >> 5);
}
// After the same exchange between registers q = 2 u and q = 2 u + 1, store h of
// pair u writes 64 contiguous bytes of 16 rows: its float from the tile's first.
__host__ __device__ inline int lsp_y_float(const LinSplitShape& S, int lane, int rt, int u, int h)
{
    return (16 * h + (lane & 15)) * S.N() + 32 * rt + 16 * u + 8 * ((lane >> 4) & 1) +
           4 * (lane >> 5);
}

// The same product in fp32: the operands of product h (two K slots) of input
// channel ci.  A lane's slot is blade jb = 2 h + lane / 32 (bitmask); MFMA row
// lane % 32 of row tile rt is output column n, whose filter blade is src_blade;
// its X row is lane % 32 of tile t, the batch's last where that lies past it.
__host__ __device__ inline int lsp_redo_j(const LinSplitShape& S, int lane, int h)
{
    return blade_perm(S.NB, 2 * h + (lane >> 5));
}
__host__ __device__ inline int lsp_redo_w(const LinSplitShape& S, int lane, int rt, int ci, int h)
{
    const int n = 32 * rt + (lane & 31);
    return lsp_w_float(S, ci, n / S.NB) + src_blade(S.NB, n % S.NB, lsp_redo_j(S, lane, h));
}
__host__ __device__ inline int64_t lsp_redo_x(const LinSplitShape& S, const LinSplitArgs& a,
                                              int64_t t, int lane, int ci, int h)
{
    const int64_t row = 32 * t + (lane & 31);
    return (row < a.B ? row : a.B - 1) * S.K() + ci * S.NB + lsp_redo_j(S, lane, h);
}

}  // namespace cliff
