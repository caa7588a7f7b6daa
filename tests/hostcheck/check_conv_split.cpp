// Host-side walk of conv_split_kernel's address arithmetic (test
// infrastructure; see check_main.cpp).  Everything below calls the kernel's
// own functions from conv_split_geom.hpp.
//
// For a launch plan it checks:
//   * launch shape: workgroup size, grid = the number of blocks, LDS bytes
//     within the 160 KiB of a CU and holding both filter slots and both input
//     buffers, every stage's input strips loaded within the stage's own steps;
//   * every workgroup (sampled on large grids): each lane's input loads for
//     the first and the last K group and every row of filter taps, and its
//     filter loads for both groups, lie inside their tensors; every output
//     store lies inside the output at the position and channel the lane holds
//     and every output multivector is stored exactly once;
//   * the LDS image of those stages: every slot a fragment read takes, for
//     every wave, lane, position tile, tap column and chunk, was written with
//     the input or filter multivector the product needs (positions and
//     channels past the end, whose results are not stored, excepted).
#include <stdlib.h>

#include <algorithm>
#include <vector>

#include "check.hpp"
#include "conv_split_geom.hpp"

namespace hostcheck {

using namespace cliff;

namespace {

template <int KD>
void walk(const LaunchPlan& p, const SplitTile& T, const SplitArgs& a)
{
    const Dims& d = current->dims;
    const Buffer* bx = find_buffer(a.x);
    const Buffer* bw = find_buffer(a.w);
    const Buffer* by = find_buffer(a.y);
    const Buffer* bb = a.bias ? find_buffer(a.bias) : nullptr;
    if (!bx || !bw || !by || (a.bias && !bb)) {
        fail("unknown buffer");
        return;
    }
    const int NB = T.NB;
    const int64_t n_x = bx->n / NB, n_w = bw->n / NB, n_y = by->n / NB;  // multivectors
    if (p.block != T.nt() || p.grid != a.n_blk || p.lds_bytes != T.lds_bytes() ||
        p.lds_bytes > 160 * 1024) {
        fail("launch shape: block %lld grid %lld lds %lld", (long long)p.block, (long long)p.grid,
             (long long)p.lds_bytes);
        return;
    }
    const int64_t n_grp = (a.C_in + T.cpg() - 1) / T.cpg();
    const int DF = p.tpl[2];
    if ((DF && DF != a.df) || a.nx > split_rounds(KD, DF) || a.xi > (DF ? 1 : 2) || (int64_t)a.xi * a.df < a.nx || a.n_step != n_grp * a.taps ||
        a.nrt * a.df != a.taps || a.nrow * a.Do != a.M || (bb && bb->n < (int64_t)a.C_out * NB)) {
        fail("stage plan: nx %d xi %d n_step %d", a.nx, a.xi, a.n_step);
        return;
    }
    // sizes the block's offsets were checked for
    int64_t D = a.D, img = 1;
    for (int t = 0; t < KD; ++t) img *= D;
    if (img != a.cin_stride || n_x < (int64_t)(a.M / a.npos) * a.C_in * img) {
        fail("input size");
        return;
    }
    const int64_t B = a.M / a.npos;
    const bool sampled = a.n_blk > 64;
    if (sampled) current->grid_sampled = true;
    std::vector<uint8_t> seen;
    const bool count = (int64_t)a.n_blk * T.pos() * T.co_wg() < (1 << 26);
    if (count) seen.assign((size_t)n_y, 0);
    const FastDiv fnpos = fast_div(a.npos);
    // multivector offset of input (m, channel 0, tap row rt, tap column qx)
    auto want_x = [&](int64_t m, int rt, int qx) {
        const int64_t b = m / a.npos;
        int64_t r = m - b * a.npos;
        int64_t c[3] = {0, 0, 0};
        for (int t = KD - 1; t >= 0; --t) {
            c[t] = r % a.Do;
            r /= a.Do;
        }
        c[KD - 1] += qx;
        if (KD == 2) c[0] += rt;
        if (KD == 3) {
            c[0] += rt / a.df;
            c[1] += rt % a.df;
        }
        int64_t o = 0;
        for (int t = 0; t < KD; ++t) o = o * D + c[t];
        return b * a.C_in * img + o;
    };
    const int SLOT = NB * 2;  // LDS bytes of one channel in one plane
    for (int64_t bi = 0; bi < a.n_blk; ++bi) {
        const SplitBlock g = split_block<KD>(T, a, (int)bi);
        if (g.m0 < 0 || g.m_end > a.M || g.m0 >= g.m_end || g.co0 < 0 || g.co0 >= a.C_out) {
            fail("block %lld: m %d..%d co %d", (long long)bi, g.m0, g.m_end, g.co0);
            return;
        }
        // outputs
        if (count)
            for (int wave = 0; wave < T.waves(); ++wave)
                for (int lane = 0; lane < 64; ++lane)
                    for (int np = 0; np < T.NPT; ++np)
                        for (int r = 0; r < T.CW / 2; ++r) {
                            const int m = split_out_m(T, g, wave, lane, np);
                            const int co = split_out_co(T, g, wave, lane, r);
                            if (m >= g.m_end || co >= a.C_out) continue;
                            const int64_t o = split_out_ofs(a, fnpos, m, co);
                            const int64_t b = m / a.npos;
                            if (o != (b * a.C_out + co) * a.npos + m % a.npos || o < 0 || o >= n_y) {
                                fail("block %lld: output %lld of %lld", (long long)bi, (long long)o,
                                     (long long)n_y);
                                return;
                            }
                            if (seen[(size_t)o]++) {
                                fail("output %lld stored twice", (long long)o);
                                return;
                            }
                        }
        // stages: all blocks of small grids, else the first, last and every 61st
        if (sampled && bi > 2 && bi + 3 < a.n_blk && bi % 61) continue;
        current->workgroups++;
        // the fp32 recompute's reads: each lane's filters, and its positions'
        // inputs at every tap (the last channel's or position's past the end)
        for (int wave = 0; wave < T.waves(); ++wave)
            for (int lane = 0; lane < 64; ++lane) {
                const int co = std::min(g.co0 + (wave % T.WCO) * T.CW + lane % T.CW, a.C_out - 1);
                const int64_t w0 = split_redo_w(T, a, g, wave, lane);
                if (w0 != (int64_t)co * a.taps ||
                    w0 + ((int64_t)(a.C_in - 1) * a.C_out + 1) * a.taps > n_w) {
                    fail("recompute reads filter %lld", (long long)w0);
                    return;
                }
                for (int np = 0; np < T.NPT; ++np) {
                    const int m = std::min(split_out_m(T, g, wave, lane, np), g.m_end - 1);
                    const int64_t x0 = g.base + split_redo_x<KD>(T, a, g, wave, lane, np);
                    for (int rt = 0; rt < a.nrt; ++rt)
                        for (int qx = 0; qx < a.df; ++qx) {
                            const int64_t x = x0 + split_rt_off<KD>(a, rt) + qx;
                            if (x != want_x(m, rt, qx) || x < 0 || x + (a.C_in - 1) * img >= n_x) {
                                fail("recompute reads input %lld of %lld (m %d rt %d qx %d)",
                                     (long long)x, (long long)n_x, m, rt, qx);
                                return;
                            }
                        }
                }
            }
        std::vector<int64_t> groups = {0};
        if (n_grp > 1) groups.push_back(n_grp - 1);
        for (int64_t gi : groups) {
            const int ci0 = (int)gi * T.cpg();
            for (int rt = 0; rt < a.nrt; ++rt) {
                if (sampled && rt && rt + 1 < a.nrt) continue;
                std::vector<int64_t> X(2 * T.x_plane() / SLOT, -1);
                for (int wave = 0; wave < T.waves(); ++wave)
                    for (int j = 0; j < a.nx; ++j)
                        for (int lane = 0; lane < 64; ++lane) {
                            const int chi = split_x_chi(T, wave), t = split_x_t(T, wave, lane, j);
                            const int64_t go = split_x_goff<KD>(a, g, t);
                            for (int c = 0; c < T.chi(); ++c) {
                                const int ci = ci0 + chi * T.chi() + c;
                                int64_t src = -2;  // zero
                                if (ci < a.C_in) {
                                    src = g.base + go + (int64_t)ci * a.cin_stride +
                                          split_rt_off<KD>(a, rt);
                                    if (src < 0 || src >= n_x) {
                                        fail("block %lld: input load %lld of %lld (t %d ci %d rt %d)",
                                             (long long)bi, (long long)src, (long long)n_x, t, ci, rt);
                                        return;
                                    }
                                }
                                if (t >= T.LP) continue;
                                const int at = split_x_lds(T, chi, t) + c * SLOT;
                                if (at < 0 || at % SLOT || at + SLOT > 2 * T.x_plane() ||
                                    X[at / SLOT] != -1) {
                                    fail("input slot %d of t %d", at, t);
                                    return;
                                }
                                X[at / SLOT] = src;
                            }
                        }
                for (int wave = 0; wave < T.waves(); ++wave)
                    for (int lane = 0; lane < 64; ++lane)
                        for (int np = 0; np < T.NPT; ++np) {
                            const int m = split_out_m(T, g, wave, lane, np);
                            const int f = split_b_frag(T, a, g, wave, lane, np);
                            for (int qx = 0; qx < a.df; ++qx)
                                for (int h = 0; h < T.cpc(); ++h) {
                                    const int at = f + qx * 16 + h * SLOT;
                                    if (at < 0 || at + SLOT > 2 * T.x_plane()) {
                                        fail("fragment at %d", at);
                                        return;
                                    }
                                    if (m >= g.m_end) continue;
                                    const int ci = ci0 + (lane >> 5) * T.cpc() + h;
                                    const int64_t want =
                                        ci < a.C_in ? want_x(m, rt, qx) + (int64_t)ci * img : -2;
                                    if (X[at / SLOT] != want) {
                                        fail("block %lld rt %d qx %d m %d ci %d: fragment holds %lld, "
                                             "not %lld", (long long)bi, rt, qx, m, ci,
                                             (long long)X[at / SLOT], (long long)want);
                                        return;
                                    }
                                }
                        }
            }
            // filters of one tap (the offset grows with the tap alone)
            std::vector<int64_t> A(2 * T.a_plane() / SLOT, -1);
            for (int e = 0; e < T.a_items() && e < T.nt(); ++e)
                for (int c = 0; c < T.chi(); ++c) {
                    const int ci = ci0 + split_a_chi(T, e) * T.chi() + c;
                    int64_t src = -2;
                    if (ci < a.C_in) {
                        src = (int64_t)ci0 * a.C_out * a.taps + split_a_goff(T, a, g, e) +
                              (int64_t)c * a.C_out * a.taps;
                        if (src < 0 || src + a.taps > n_w) {
                            fail("filter load %lld of %lld", (long long)src, (long long)n_w);
                            return;
                        }
                    }
                    const int at = split_a_lds(T, e) + c * SLOT;
                    if (at < 0 || at % SLOT || at + SLOT > 2 * T.a_plane() || A[at / SLOT] != -1) {
                        fail("filter slot %d", at);
                        return;
                    }
                    A[at / SLOT] = src;
                }
            for (int wave = 0; wave < T.waves(); ++wave)
                for (int lane = 0; lane < 64; ++lane)
                    for (int h = 0; h < T.cpc(); ++h) {
                        // row (lane % 32) / CW of the row tile: its pair of planes
                        const int at = split_a_frag(T, wave, lane) + h * SLOT -
                                       (split_a_plane(T, 0, (lane & 31) / T.CW, 0) -
                                        split_a_plane(T, 0, 0, 0));
                        const int ci = ci0 + (lane >> 5) * T.cpc() + h;
                        // MFMA row lane % 32 holds output channel row % CW of the wave
                        const int co = g.co0 + (wave % T.WCO) * T.CW + (lane & 31) % T.CW;
                        if (at < 0 || at + SLOT > 2 * T.a_plane()) {
                            fail("filter fragment at %d", at);
                            return;
                        }
                        if (co >= a.C_out) continue;
                        const int64_t want =
                            ci < a.C_in ? ((int64_t)ci * a.C_out + co) * a.taps : -2;
                        if (A[at / SLOT] != want) {
                            fail("filter fragment co %d ci %d holds %lld, not %lld", co, ci,
                                 (long long)A[at / SLOT], (long long)want);
                            return;
                        }
                    }
        }
    }
    // planes lie one behind the other inside a slot or buffer
    if (split_a_plane(T, 2, NB - 1, 1) + T.a_plane() != T.a_bytes() ||
        split_x_plane(T, 2, 1) + T.x_plane() != T.x_bytes())
        fail("plane offsets");
    if (count) {
        const int64_t n = B * a.C_out * a.npos;
        for (int64_t o = 0; o < n; ++o)
            if (!seen[(size_t)o]) {
                fail("output %lld never stored", (long long)o);
                return;
            }
    }
    (void)d;
}

}  // namespace

void check_conv_split(const LaunchPlan& p)
{
    const SplitArgs& a = *static_cast<const SplitArgs*>(p.args);
    // tpl[2]: the unrolled filter length, 0 for any
    const SplitTile T{p.tpl[0], p.tpl[1], p.tpl[3], p.tpl[4], p.tpl[5], p.tpl[6], p.tpl[7]};
    if (T.KD == 1) walk<1>(p, T, a);
    if (T.KD == 2) walk<2>(p, T, a);
    if (T.KD == 3) walk<3>(p, T, a);
}

}  // namespace hostcheck
