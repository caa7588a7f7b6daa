// Host-side walk of linear_split_kernel's address arithmetic (test
// infrastructure; see check_main.cpp), through the kernel's own functions from
// linear_split_geom.hpp: launch shape and LDS size; every weight item's reads
// inside the weight and every LDS slot written once; every fragment read of
// every lane at the slot of its row and K chunk; and for every tile (sampled
// past 2^15) the input loads of each lane inside the tile's descriptor and at
// the row and K values of the chunk, and every output float4 inside the
// descriptor stored once, at the lane's row, with none of a row past B.
#include <algorithm>
#include <vector>

#include "check.hpp"
#include "linear_split_geom.hpp"

namespace hostcheck {

using namespace cliff;

void check_linear_split(const LaunchPlan& p)
{
    const LinSplitArgs& a = *static_cast<const LinSplitArgs*>(p.args);
    const LinSplitShape S{p.tpl[0], p.tpl[1], p.tpl[2]};
    const int PF = p.tpl[3], N = S.N(), K = S.K();
    const Buffer *bx = find_buffer(a.x), *bw = find_buffer(a.w), *by = find_buffer(a.y);
    const Buffer* bb = a.bias ? find_buffer(a.bias) : nullptr;
    if (!bx || !bw || !by || (a.bias && (!bb || bb->n < N))) {
        fail("unknown buffer");
        return;
    }
    if (a.C_out * S.NB != N || a.C_in * S.NB != K || bx->n < a.B * K || by->n < a.B * N ||
        a.n_tile != (a.B + 31) / 32 || p.block != 512 || p.grid < 1 ||
        p.grid > std::max<int64_t>((a.n_tile + 7) / 8, 1) || p.lds_bytes != S.lds_bytes() ||
        p.lds_bytes > 160 * 1024 || PF < 1 || S.KQ % PF) {
        fail("launch shape");
        return;
    }
    // weight: LDS image of (chunk, column) -> item's channel and chunk
    std::vector<int> img((size_t)S.plane() / 16, -1);
    for (int e = 0; e < S.items(); ++e) {
        const int co = lsp_w_co(S, e), chunk = lsp_w_chunk(S, e);
        for (int u = 0; u < 8; ++u) {
            const int64_t f = lsp_w_float(S, (8 * chunk + u) / S.NB, co) + u % S.NB;
            const int64_t want =
                ((int64_t)((8 * chunk + u) / S.NB) * a.C_out + co) * S.NB + u % S.NB;
            if (f != want || f < 0 || f >= bw->n) {
                fail("weight read %lld of %lld", (long long)f, (long long)bw->n);
                return;
            }
        }
        for (int i = 0; i < S.NB; ++i) {
            const int at = lsp_a_byte(S, chunk, co * S.NB + i);
            if (at < 0 || at % 16 || at + 16 > S.plane() || img[at / 16] != -1) {
                fail("weight slot %d", at);
                return;
            }
            img[at / 16] = chunk * N + co * S.NB + i;
        }
    }
    for (int lane = 0; lane < 64; ++lane)
        for (int s = 0; s < S.KQ; ++s)
            for (int r = 0; r < S.RT; ++r) {
                const int at = lsp_a_byte(S, lane >> 5, lane & 31) + lsp_a_byte(S, 2 * s, 32 * r);
                if (at < 0 || at + 16 > S.plane() ||
                    img[at / 16] != (2 * s + (lane >> 5)) * N + 32 * r + (lane & 31)) {
                    fail("fragment of lane %d step %d row tile %d", lane, s, r);
                    return;
                }
            }
    // the fp32 recompute's weight reads: product h of input channel ci puts blade
    // 2 h + lane / 32 into K slot lane / 32
    for (int lane = 0; lane < 64; ++lane)
        for (int r = 0; r < S.RT; ++r)
            for (int ci = 0; ci < a.C_in; ++ci)
                for (int h = 0; h < S.NB / 2; ++h) {
                    const int n = 32 * r + (lane & 31), jb = 2 * h + (lane >> 5);
                    const int ib = blade_perm(S.NB, n % S.NB);
                    const int64_t want = ((int64_t)ci * a.C_out + n / S.NB) * S.NB +
                                         blade_perm(S.NB, ib ^ jb);
                    if (lsp_redo_w(S, lane, r, ci, h) != want || want >= bw->n ||
                        lsp_redo_j(S, lane, h) != blade_perm(S.NB, jb)) {
                        fail("recompute reads weight %d", lsp_redo_w(S, lane, r, ci, h));
                        return;
                    }
                }
    const bool sampled = a.n_tile > (1 << 15);
    if (sampled) current->grid_sampled = true;
    std::vector<uint8_t> seen((size_t)N * 32);
    for (int64_t t = 0; t < a.n_tile; ++t) {
        if (sampled && t > 2 && t + 3 < a.n_tile && t % 997) continue;
        const int rows = lsp_rows(a, t);
        if (rows < 1 || 32 * t + rows > a.B) {
            fail("tile %lld has %d rows", (long long)t, rows);
            return;
        }
        std::fill(seen.begin(), seen.end(), 0);
        for (int lane = 0; lane < 64; ++lane) {
            for (int ci = 0; ci < a.C_in; ++ci)
                for (int h = 0; h < S.NB / 2; ++h) {
                    const int64_t row = std::min<int64_t>(32 * t + (lane & 31), a.B - 1);
                    const int64_t want =
                        row * K + ci * S.NB + blade_perm(S.NB, 2 * h + (lane >> 5));
                    if (lsp_redo_x(S, a, t, lane, ci, h) != want || want < 0 || want >= bx->n) {
                        fail("recompute reads input %lld", (long long)want);
                        return;
                    }
                }
            // (the kernel adds 64 s + 16 rows h to its first offset)
            for (int s = 0; s < S.KQ; ++s)
                for (int h = 0; h < 2; ++h) {
                    const int off = lsp_x_float(S, lane, 0, 0) +
                                    (lsp_x_float(S, 0, 0, 1) - lsp_x_float(S, 0, 0, 0)) * h + 16 * s;
                    if (off != lsp_x_float(S, lane, s, h) || off < 0 || off + 4 > 32 * K) {
                        fail("input load %d", off);
                        return;
                    }
                    // after the exchange: which lane and register holds it
                    const int row = off / K, k = off % K, lr = lane >> 4;
                    const int to = (lr & 1) == h ? lane : lane ^ 16;
                    const int reg = (lr & 1) == h ? h : h ^ 1;
                    if ((to & 31) != row || k != 16 * s + 8 * (to >> 5) + 4 * reg) {
                        fail("lane %d register %d holds row %d K %d", to, reg, row, k);
                        return;
                    }
                }
            for (int r = 0; r < S.RT; ++r)
                for (int u = 0; u < 2; ++u)
                    for (int h = 0; h < 2; ++h) {
                        // value of accumulator pair register h of this lane, and
                        // the store that takes it after the exchange
                        const int lr = lane >> 4;
                        const int to = (lr & 1) == h ? lane : lane ^ 16;
                        const int reg = (lr & 1) == h ? h : h ^ 1;
                        const int want = (lane & 31) * N + lsp_y_col(S, lane, r, 2 * u + h);
                        const int at = lsp_y_float(S, to, r, u, reg);
                        if (at != want || at < 0 || at % 4 || at + 4 > 32 * N) {
                            fail("output float %d, not %d", at, want);
                            return;
                        }
                        for (int e = 0; e < 4; ++e)
                            if (seen[at + e]++) {
                                fail("output %d of tile %lld stored twice", at + e, (long long)t);
                                return;
                            }
                    }
        }
        for (size_t i = 0; i < seen.size(); ++i)
            if (!seen[i]) {
                fail("output %zu of a tile never stored", i);
                return;
            }
        current->workgroups++;
    }
}

}  // namespace hostcheck
