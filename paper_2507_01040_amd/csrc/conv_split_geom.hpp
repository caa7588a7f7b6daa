// Address arithmetic of conv_split_kernel: which input values and filters a
// workgroup stages, where they land in LDS, which LDS bytes each MFMA fragment
// reads and where each output goes.  The kernel and the host-side bounds
// checker (a CPU build of the library used by the tests) both call these
// functions, so the checker verifies the kernel's own arithmetic.
#pragma once

#include <stdint.h>

#include "common.hpp"
#include "conv_mfma_geom.hpp"

namespace cliff {

struct SplitArgs {
    const float* x;
    const float* w;
    const float* bias;
    float* y;
    int C_in, C_out, D, Do, df;
    int M;        // number of output positions B * d_out^k
    int npos;     // d_out^k
    int nrow;     // output rows M / d_out
    int taps;     // d_filter^k
    int nrt;      // rows of filter taps: d_filter^(k - 1)
    int n_step;   // groups of input channels * nrt * d_filter
    int n_co_blk, n_blk;
    int nx, xi;   // strip rounds of a stage's input, and those of one step
    int cin_stride;  // d_image^k: multivectors between input channels
    SignMasks sign;
    uint32_t sx[32], sz[32];  // sign bits and keep masks of two K slots, [i][pair]
    ActParams act;
};

// The compile-time shape of one kernel instantiation.  KD spatial dimensions,
// NB blades; WCO x WPOS waves, each CW output channels (32 or 16) by 32 * NPT
// positions; LP input positions staged per K group.  A wave holds a row of CW
// output channels for each of the NB output blades; 32 / CW of them fill an
// MFMA row tile.
struct SplitTile {
    int KD, NB, WCO, WPOS, NPT, LP, CW = 32;
    __host__ __device__ constexpr int rpt() const { return 32 / CW; }  // rows of a row tile
    __host__ __device__ constexpr int waves() const { return WCO * WPOS; }
    __host__ __device__ constexpr int nt() const { return 64 * waves(); }
    __host__ __device__ constexpr int co_wg() const { return CW * WCO; }
    __host__ __device__ constexpr int pos() const { return 32 * NPT * WPOS; }
    // input channels of one K group (16 slots), of one 8-slot chunk, and of
    // one lane's conversion item (8 slots at most, 8 filter floats at most)
    __host__ __device__ constexpr int cpg() const { return 16 / NB; }
    __host__ __device__ constexpr int cpc() const { return 8 / NB; }
    __host__ __device__ constexpr int chi() const { return NB == 2 ? 2 : 1; }
    __host__ __device__ constexpr int nchi() const { return cpg() / chi(); }
    __host__ __device__ constexpr int a_items() const { return co_wg() * nchi(); }
    // LDS bytes: two filter slots (one K group of one tap), two input buffers
    __host__ __device__ constexpr int a_plane() const { return co_wg() * 16; }
    __host__ __device__ constexpr int a_bytes() const { return 3 * NB * 2 * a_plane(); }
    __host__ __device__ constexpr int x_plane() const { return LP * 16; }
    __host__ __device__ constexpr int x_bytes() const { return 3 * 2 * x_plane(); }
    __host__ __device__ constexpr int lds_bytes() const { return 2 * (a_bytes() + x_bytes()); }
};

// The most strip rounds of a stage: one for each of the DF tap columns where
// their number is fixed, else what a lane keeps offsets for.
__host__ __device__ constexpr int split_rounds(int KD, int DF) { return DF > 0 ? DF : KD == 1 ? 8 : 4; }

// LDS byte offsets of the planes: term t (0 high, 1 middle, 2 low part), row
// (output blade) r, chunk g of 8 K slots.
__host__ __device__ constexpr int split_a_plane(const SplitTile& T, int t, int r, int g)
{
    return ((t * T.NB + r) * 2 + g) * T.a_plane();
}
__host__ __device__ constexpr int split_x_plane(const SplitTile& T, int t, int g)
{
    return (t * 2 + g) * T.x_plane();
}

// One workgroup's block: P consecutive flattened output positions [m0, m_end)
// by CO_WG output channels from co0.  Its input, for one row of filter taps,
// is a run of positions in the concatenated input rows of the output rows it
// touches: run index t is column (x0 + t) mod d_image of row
// row0 + (x0 + t) / d_image.
struct SplitBlock {
    int co0, m0, m_end, row0, x0;
    int64_t base;  // multivector offset of (row0, column 0), channel 0, tap 0
    FastDiv fD, fDo;
};

// Multivector offset (channel 0, tap row 0, column 0) of output row `row`.
template <int KD>
__host__ __device__ inline int64_t split_row_base(const SplitArgs& a, const FastDiv& fDo, int row)
{
    const int64_t D = a.D;
    if (KD == 1) return (int64_t)row * a.C_in * D;
    const int q = fdiv(row, fDo), r = row - q * a.Do;
    if (KD == 2) return (int64_t)q * a.C_in * D * D + r * D;
    const int b = fdiv(q, fDo), z = q - b * a.Do;
    return (int64_t)b * a.C_in * D * D * D + (z * D + r) * D;
}

template <int KD>
__host__ __device__ inline SplitBlock split_block(const SplitTile& T, const SplitArgs& a, int bid)
{
    SplitBlock g;
    // Workgroups are dispatched round-robin over the 8 XCDs; renumbered so
    // each XCD (own L2) works through a contiguous run of position blocks.
    const int per = a.n_blk >> 3, rem = a.n_blk & 7;
    const int xcd = bid & 7, slot = bid >> 3;
    const int tile = xcd < rem ? xcd * (per + 1) + slot
                               : rem * (per + 1) + (xcd - rem) * per + slot;
    const int pos_blk = udiv(tile, a.n_co_blk);
    g.co0 = (tile - pos_blk * a.n_co_blk) * T.co_wg();
    const int P = T.pos();
    g.m0 = pos_blk * P;
    g.m_end = P < a.M - g.m0 ? g.m0 + P : a.M;
    g.fD = fast_div(a.D);
    g.fDo = fast_div(a.Do);
    g.row0 = fdiv(g.m0, g.fDo);
    g.x0 = g.m0 - g.row0 * a.Do;
    g.base = split_row_base<KD>(a, g.fDo, g.row0);
    return g;
}

// Run index of a lane's output position (tap column 0); positions past the
// end read the last one's input.
__host__ __device__ inline int split_run(const SplitArgs& a, const SplitBlock& g, int m)
{
    const int mc = m < g.m_end ? m : g.m_end - 1;
    const int row = fdiv(mc, g.fDo);
    return (row - g.row0) * a.D + (mc - row * a.Do) - g.x0;
}

// Input item of one wave and round: channels chi * CHI ... of the K group at
// run index t (a strip of 64 positions per wave and round).
__host__ __device__ inline int split_x_chi(const SplitTile& T, int wave) { return wave % T.nchi(); }
__host__ __device__ inline int split_x_t(const SplitTile& T, int wave, int lane, int j)
{
    return (j * (T.waves() / T.nchi()) + wave / T.nchi()) * 64 + lane;
}
// Its offset in multivectors from the block's base, for channel 0 and tap row
// 0 (rows past the last output row are read from it; never multiplied into a
// stored output).
template <int KD>
__host__ __device__ inline int split_x_goff(const SplitArgs& a, const SplitBlock& g, int t)
{
    const int u = g.x0 + t, row = fdiv(u, g.fD), x = u - row * a.D;
    const int r = g.row0 + row < a.nrow ? g.row0 + row : a.nrow - 1;
    return (int)(split_row_base<KD>(a, g.fDo, r) - g.base) + x;
}
// Multivectors from tap row 0 to tap row rt (k = 3: qz * d_filter + qy).
template <int KD>
__host__ __device__ inline int split_rt_off(const SplitArgs& a, int rt)
{
    if (KD == 1) return 0;
    if (KD == 2) return rt * a.D;
    const int qz = udiv(rt, a.df);
    return (qz * a.D + (rt - qz * a.df)) * a.D;
}
// LDS byte of an item's slots inside the plane group of one term: add
// split_x_plane(term, 0).
__host__ __device__ inline int split_x_lds(const SplitTile& T, int chi, int t)
{
    const int ch = chi * T.chi();
    return (ch / T.cpc()) * T.x_plane() + t * 16 + (ch % T.cpc()) * T.NB * 2;
}

// Filter item: output channel co0 + e % CO_WG, channels (e / CO_WG) * CHI ...
// of the K group.
__host__ __device__ inline int split_a_co(const SplitTile& T, int e) { return e % T.co_wg(); }
__host__ __device__ inline int split_a_chi(const SplitTile& T, int e) { return e / T.co_wg(); }
// Multivector offset from the filters of (first channel of the group, channel
// co 0, tap): rows past C_out read the last channel's (never stored).
__host__ __device__ inline int split_a_goff(const SplitTile& T, const SplitArgs& a,
                                            const SplitBlock& g, int e)
{
    const int co = g.co0 + split_a_co(T, e);
    const int cc = co < a.C_out ? co : a.C_out - 1;
    return (split_a_chi(T, e) * T.chi() * a.C_out + cc) * a.taps;
}
__host__ __device__ inline int split_a_lds(const SplitTile& T, int e)
{
    const int ch = split_a_chi(T, e) * T.chi();
    return (ch / T.cpc()) * T.a_plane() + split_a_co(T, e) * 16 + (ch % T.cpc()) * T.NB * 2;
}

// MFMA fragment reads of a lane (add the plane of the term, and the row's).
// MFMA row lane % 32 of a row tile is output channel lane % CW of the wave, in
// row (lane % 32) / CW of the tile's.
__host__ __device__ inline int split_a_frag(const SplitTile& T, int wave, int lane)
{
    return ((lane & 31) / T.CW * 2 + (lane >> 5)) * T.a_plane() +
           ((wave % T.WCO) * T.CW + lane % T.CW) * 16;
}
__host__ __device__ inline int split_b_frag(const SplitTile& T, const SplitArgs& a,
                                            const SplitBlock& g, int wave, int lane, int np)
{
    const int m = g.m0 + ((wave / T.WCO) * T.NPT + np) * 32 + (lane & 31);
    return (lane >> 5) * T.x_plane() + split_run(a, g, m) * 16;
}

// The same product in fp32 (split_fp32_sums): multivector offset of the filters
// of MFMA row lane % 32 (channel 0, tap 0) and, from the block's base, of the
// input of column tile np (channel 0, tap 0), both of the last channel or
// position where the lane's own is past the end.
__host__ __device__ inline int64_t split_redo_w(const SplitTile& T, const SplitArgs& a,
                                                const SplitBlock& g, int wave, int lane)
{
    const int co = g.co0 + (wave % T.WCO) * T.CW + lane % T.CW;
    return (int64_t)(co < a.C_out ? co : a.C_out - 1) * a.taps;
}
template <int KD>
__host__ __device__ inline int split_redo_x(const SplitTile& T, const SplitArgs& a,
                                            const SplitBlock& g, int wave, int lane, int np)
{
    const int m = g.m0 + ((wave / T.WCO) * T.NPT + np) * 32 + (lane & 31);
    return split_x_goff<KD>(a, g, split_run(a, g, m));
}

// Output channel of accumulator register r (0..CW / 2 - 1, of a row tile's first
// row) and position of column tile np of a lane.
__host__ __device__ inline int split_out_co(const SplitTile& T, const SplitBlock& g, int wave,
                                            int lane, int r)
{
    return g.co0 + (wave % T.WCO) * T.CW + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
}
__host__ __device__ inline int split_out_m(const SplitTile& T, const SplitBlock& g, int wave,
                                           int lane, int np)
{
    return g.m0 + ((wave / T.WCO) * T.NPT + np) * 32 + (lane & 31);
}
// Multivector offset of output (m, co).
__host__ __device__ inline int64_t split_out_ofs(const SplitArgs& a, const FastDiv& fnpos, int m,
                                                 int co)
{
    const int b = fdiv(m, fnpos);
    return ((int64_t)b * a.C_out + co) * a.npos + (m - b * a.npos);
}

}  // namespace cliff
