// k-D Clifford convolution (paper, Algorithm 1) on the bf16 matrix cores with
// fp32 accuracy: every fp32 operand is the exact sum of three bf16 parts, and
// every product of two operands six products of parts, summed in fp32 by
// v_mfma_f32_32x32x16_bf16.
//
// Parts.  h = bf16(v), m = bf16(v - h), l = bf16(v - h - m), rounded to
// nearest, of v = 2^16 times the operand (split.hpp): v = h + m + l to the last
// bit, for every float below 2^112.  The products h h, h m, m h, m m, h l, l h
// are kept; those left out are below 2^-24 of the operands' product.
//
// Row i of an MFMA tile's rows is output blade i, and the K slots of an input
// channel are its blades j with filter blade i ^ j and the table's sign, so
// every product of two blades is taken by itself and a blade's sum never meets
// another blade's.  For g = (1, 1), (1, -1), (-1, 1) and (1, 1, 1) the products
// of 2 x 2 matrices would be half as many (k = 2, C 64, d 128 342 us), but their
// elements are sums of blades, rounded in fp32: beside a blade 1e4 times as
// large a blade's output kept two digits.  Any scheme of fewer products adds
// blades, and no more parts help the accumulators that hold the sums.
//
// Work decomposition.  P consecutive flattened output positions by CO_WG
// output channels per workgroup.  The K loop runs over steps: one group of 16
// K slots (16 / N_B input channels) of one filter tap.  The three parts of the
// step's filters lie in an LDS ring of two slots, those of the input in two
// buffers, one per stage (K group and row of filter taps: the taps of a row
// read the same run of positions at a shift).  During a step each lane loads
// the raw fp32 filters of the next step and a strip of the next stage's input,
// converts them after the step's MFMAs and writes the parts to the other slot
// and buffer; one barrier per step.
//
// 16 channels (CW).  An MFMA row tile holds 32 channels of one output blade, or
// 16 channels of two: the lane that has (channel, position) then finds the
// second one eight registers on.  k = 2 layers of up to 16 channels, or of a
// last block of up to 16, ran half of their MFMAs on padding: B 8, C 16, d 258
// 342 -> 193 us (fp32 tiles: 289; with a gate 218 and 299).  The staging and the
// barrier of a step stay, so wider layers keep 32.
//
// Bound: the bf16 matrix cores at the clock their power allows.  A loop of
// 32x32x16 MFMAs on random registers reaches 1793 TFLOP/s (2485 on zeros);
// this kernel's MFMAs run at 1270 (k = 3, C 32, d 32) to 1460 TFLOP/s (k = 2,
// C 64, d 128; k = 3, C 64, d 36), busy 61 to 77 % of the cycles; the rest is
// staging, the barrier and the first fragments' reads.  Measured against the
// fp32 tiles: k = 2, B 8, C 64, d 128, 3x3 1078 -> 615 us; k = 3, B 8, C 32, d 32
// 5.43 -> 3.62 ms; C 64, d 36 30.9 -> 18.3 ms; k = 1, B 4096, C 64, d 60, 17 taps
// 712 -> 516 us.  The error against 64 bits falls from 8.6e-7 to 7.4e-7 (2-norm,
// 2304 products), as 16 products go into one rounding; where products are zero,
// which the fp32 tiles do not round, it stays: vector-valued inputs 6.1e-7 -> 7.1e-7
// (k = 3: 1.33 times the fp32 tiles'), inputs of one blade 1.2 to 2.0 times.
// Tried on the 2 x 2 matrix form: 16x16x32 MFMAs with two products of parts in
// one (2055 TFLOP/s on registers, but 28 instead of 18 KB of LDS reads a step
// and spills: 360 -> 428 us at k = 2), a third filter slot with fragments read
// ahead of the barrier (335 -> 349 us), loads right after the conversions
// instead of at the start of a step (360 -> 397 us), all taps of a row loaded at
// once (360 -> 369 us).
//
// Values that bf16 arithmetic cannot carry (infinities, operands from 2^112 and
// sums from 2^96 on) come out non-finite; a wave that holds such a sum computes
// all of its sums again on the fp32 matrix cores (split_fp32_sums).  With a channel
// of the lowest value in all images but one C 64, d 128 takes 1.8 ms (fp32 tiles 1.1;
// one lane for an output, half of the images masked: 16), k = 1, B 1024, C 64,
// d 60, 17 taps 0.57 ms (0.21; 7.3), k = 3, C 32, d 32, B 2 2.8 ms (1.4; 95).
#include <stdio.h>

#include <algorithm>
#include <cmath>

#include "common.hpp"
#include "conv_split_geom.hpp"
#include "epilogue.hpp"
#include "split.hpp"

namespace cliff {
namespace {

typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f16 __attribute__((ext_vector_type(16)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

// A wave's accumulators as sums of fp32 products on the fp32 matrix cores, for
// values that bf16 parts cannot hold: operands straight from memory, one tap of
// one input channel at a time and the next one's loads ahead of it.
template <int KD, int NB, int R, int NPT>
__device__ void split_fp32_sums(const SplitTile& T, const SplitArgs& a, const SplitBlock& g,
                                int wave, int lane, f16 (&acc)[R][NPT])
{
    constexpr int RPT = NB / R;
    // MFMA row lane % 32 is output blade RPT r + hi, K slot lane / 32 of product
    // h input blade 2 h + jl (bitmasks): filter blade (RPT r ^ 2 h) ^ hi ^ jl
    const int hi = (lane & 31) / T.CW, jl = lane >> 5;
    const bool odd = hi ^ jl;
    float sg[R][NB / 2];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int h = 0; h < NB / 2; ++h)
            sg[r][h] = sign_of(a.sign, blade_perm(NB, RPT * r + hi) * NB + blade_perm(NB, 2 * h + jl));
    const float* const wp = a.w + split_redo_w(T, a, g, wave, lane) * NB;
    const float* xp[NPT];
#pragma unroll
    for (int np = 0; np < NPT; ++np)
        xp[np] = a.x + (g.base + split_redo_x<KD>(T, a, g, wave, lane, np)) * NB;
    auto load = [&](const float* p, float (&v)[NB]) {
        if constexpr (NB == 2) {
            const f2 q = *reinterpret_cast<const f2*>(p);
            v[0] = q[0];
            v[1] = q[1];
        } else {
#pragma unroll
            for (int h = 0; h < NB / 4; ++h) {
                const f4 q = reinterpret_cast<const f4*>(p)[h];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * h + e] = q[e];
            }
        }
    };
    // PD taps in flight: the few products of small multivectors do not cover a
    // load's latency
    constexpr int PD = NB == 2 ? 4 : NB == 4 ? 2 : 1;
    float w[PD][NB], x[PD][NPT][NB];
    int ci = 0, rt = 0, qx = 0;  // the tap to be loaded next
    auto load_tap = [&](float (&wt)[NB], float (&xt)[NPT][NB]) {
        if (ci >= a.C_in) return;
        const int64_t xo = (int64_t)ci * a.cin_stride + split_rt_off<KD>(a, rt) + qx;
        load(wp + ((int64_t)ci * a.C_out * a.taps + rt * a.df + qx) * NB, wt);
#pragma unroll
        for (int np = 0; np < NPT; ++np) load(xp[np] + xo * NB, xt[np]);
        if (++qx == a.df) {
            qx = 0;
            if (++rt == a.nrt) {
                rt = 0;
                ++ci;
            }
        }
    };
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int np = 0; np < NPT; ++np)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[r][np][e] = 0.f;
#pragma unroll
    for (int d = 0; d < PD; ++d) load_tap(w[d], x[d]);
    const int n = a.C_in * a.taps;
    for (int t0 = 0; t0 < n; t0 += PD)
#pragma unroll
        for (int d = 0; d < PD; ++d) {
            if (t0 + d >= n) break;
            float wo[NB], xo[NPT][NB / 2];
#pragma unroll
            for (int e = 0; e < NB; ++e)
                wo[e] = odd ? w[d][blade_perm(NB, e ^ 1)] : w[d][blade_perm(NB, e)];
#pragma unroll
            for (int np = 0; np < NPT; ++np)
#pragma unroll
                for (int h = 0; h < NB / 2; ++h)
                    xo[np][h] =
                        jl ? x[d][np][blade_perm(NB, 2 * h + 1)] : x[d][np][blade_perm(NB, 2 * h)];
            load_tap(w[d], x[d]);
#pragma unroll
            for (int h = 0; h < NB / 2; ++h)
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const float f = sg[r][h] * wo[(RPT * r) ^ (2 * h)];
#pragma unroll
                    for (int np = 0; np < NPT; ++np)
                        acc[r][np] =
                            __builtin_amdgcn_mfma_f32_32x32x2f32(f, xo[np][h], acc[r][np], 0, 0, 0);
                }
        }
}

template <int KD, int NB, int DF, int WCO, int WPOS, int NPT, int LP, int CW>
__global__ __launch_bounds__(64 * WCO * WPOS, 2) void conv_split_kernel(SplitArgs a)
{
    constexpr SplitTile T{KD, NB, WCO, WPOS, NPT, LP, CW};
    constexpr int RPT = T.rpt(), R = NB / RPT, CHI = T.chi();
    constexpr int NT = T.nt();
    constexpr int NXMAX = split_rounds(KD, DF);  // strip rounds of a stage

    extern __shared__ u4 smem4[];
    char* smem = reinterpret_cast<char*>(smem4);
    char* const la = smem;
    char* const lx = smem + 2 * T.a_bytes();

    const SplitBlock g = split_block<KD>(T, a, blockIdx.x);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // conversion items of this lane: input strips (byte offset from the
    // block's base, LDS byte), one filter item
    const int xchi = split_x_chi(T, wave);
    int xgoff[NXMAX], xlds[NXMAX];
#pragma unroll
    for (int j = 0; j < NXMAX; ++j) {
        const int t = split_x_t(T, wave, lane, j);
        xgoff[j] = j < a.nx ? split_x_goff<KD>(a, g, t) * (NB * 4) : 0;
        xlds[j] = split_x_lds(T, xchi, t);
    }
    const bool a_on = T.a_items() >= NT || tid < T.a_items();
    const int agoff = a_on ? split_a_goff(T, a, g, tid) * (NB * 4) : 0;
    const int a_chan = a.C_out * a.taps * (NB * 4);  // bytes between input channels
    char* const aw = la + split_a_lds(T, tid);
    const float* const xbase = a.x + g.base * NB;

    // K position of a stage: first channel of the group, tap row
    struct Pos {
        int ci0, rt;
    };
    // the next stage; after the last one the last again (loaded, never used)
    auto next_stage = [&](const Pos& p) {
        Pos q{p.ci0, p.rt + 1};
        if (q.rt == a.nrt) {
            q.rt = 0;
            q.ci0 += T.cpg();
        }
        return q.ci0 < a.C_in ? q : p;
    };

    // Loads go through buffer descriptors: channels past C_in get an offset
    // (or a size) that the hardware answers with zeros, without a branch.
    auto load_mv = [&](__amdgpu_buffer_rsrc_t d, int off, int imm, float (&v)[NB]) {
        if constexpr (NB == 2) {
            const f2 q =
                __builtin_bit_cast(f2, __builtin_amdgcn_raw_buffer_load_b64(d, off, imm, 0));
            v[0] = q[0];
            v[1] = q[1];
        } else {
#pragma unroll
            for (int h = 0; h < NB / 4; ++h) {
                const f4 q = __builtin_bit_cast(
                    f4, __builtin_amdgcn_raw_buffer_load_b128(d, off + 16 * h, imm, 0));
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * h + e] = q[e];
            }
        }
    };
    // raw filters of one step, `off` bytes from channel 0's first tap; the
    // channels past C_in lie past the tensor's end
    const __amdgpu_buffer_rsrc_t wdesc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(a.w), (short)0, a.C_in * a_chan, 0x00020000);
    auto load_a = [&](int off, float (&v)[CHI][NB]) {
#pragma unroll
        for (int c = 0; c < CHI; ++c) load_mv(wdesc, agoff + (off + c * a_chan), 0, v[c]);
    };
    auto write_slots = [&](char* p, const uint32_t* d) {  // CHI * NB slots of one plane
        if constexpr (CHI * NB == 4)
            *reinterpret_cast<u2*>(p) = u2{d[0], d[1]};
        else
            *reinterpret_cast<u4*>(p) = u4{d[0], d[1], d[2], d[3]};
    };
    auto store_a = [&](int slot, const float (&ra)[CHI][NB]) {
        if (!a_on) return;
        char* const p = aw + slot;
        // K slots in bitmask order; row i takes blade i ^ j for slot j
        constexpr int NP = NB / 2;
        Parts s[CHI][NP];
#pragma unroll
        for (int c = 0; c < CHI; ++c)
#pragma unroll
            for (int h = 0; h < NP; ++h)
                s[c][h] = split2(ra[c][blade_perm(NB, 2 * h)], ra[c][blade_perm(NB, 2 * h + 1)]);
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                uint32_t d[CHI * NP];
#pragma unroll
                for (int c = 0; c < CHI; ++c)
#pragma unroll
                    for (int h = 0; h < NP; ++h) {
                        uint32_t v = s[c][h ^ (i >> 1)].t[t];
                        if (i & 1) v = __builtin_amdgcn_alignbit(v, v, 16);
                        d[c * NP + h] = (v ^ a.sx[i * NP + h]) & a.sz[i * NP + h];
                    }
                write_slots(p + split_a_plane(T, t, i, 0), d);
            }
    };
    // raw input of one strip of a stage (tap column 0); channels past C_in
    // have a descriptor of size zero, which reads zeros
    struct XDesc {
        __amdgpu_buffer_rsrc_t d[CHI];
    };
    auto x_desc = [&](const Pos& p) {
        XDesc r;
        const int64_t rt = split_rt_off<KD>(a, p.rt);
#pragma unroll
        for (int c = 0; c < CHI; ++c) {
            const int ci = p.ci0 + xchi * CHI + c;
            const float* xs = xbase + ((int64_t)ci * a.cin_stride + rt) * NB;
            r.d[c] = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(xs), (short)0,
                                                       ci < a.C_in ? 0x7fffffff : 0, 0x00020000);
        }
        return r;
    };
    auto load_x = [&](const XDesc& r, int goff, float (&v)[CHI][NB]) {
#pragma unroll
        for (int c = 0; c < CHI; ++c) load_mv(r.d[c], goff, 0, v[c]);
    };
    auto store_x = [&](int buf, int lds, bool on, const float (&v)[CHI][NB]) {
        if (!on) return;
        char* const p = lx + buf + lds;
        constexpr int NP = NB / 2;
        Parts s[CHI * NP];
#pragma unroll
        for (int c = 0; c < CHI; ++c)
#pragma unroll
            for (int h = 0; h < NP; ++h)
                s[c * NP + h] =
                    split2(v[c][blade_perm(NB, 2 * h)], v[c][blade_perm(NB, 2 * h + 1)]);
#pragma unroll
        for (int t3 = 0; t3 < 3; ++t3) {
            uint32_t d[CHI * NP];
#pragma unroll
            for (int h = 0; h < CHI * NP; ++h) d[h] = s[h].t[t3];
            write_slots(p + split_x_plane(T, t3, 0), d);
        }
    };

    f16 acc[R][NPT];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int n = 0; n < NPT; ++n)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[r][n][e] = 0.f;

    const char* const fa0 = la + split_a_frag(T, wave, lane);
    const char* fb0[NPT];
#pragma unroll
    for (int np = 0; np < NPT; ++np) fb0[np] = lx + split_b_frag(T, a, g, wave, lane, np);

    auto frag = [&](const char* p) { return *reinterpret_cast<const b8*>(p); };
    // The six products of parts, smallest first.
    constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
    // One step's MFMAs, in regions of one streamed fragment (a column tile's,
    // or a row's) by all held ones.  Within a region the next fragment's LDS
    // reads are spread between the MFMAs; `load()`, the next step's global
    // loads, goes behind the first fragments' reads, and `convert(0)` and
    // `convert(1)`, the vector work on them, between the MFMAs of the last two
    // regions.
    constexpr bool HOLD_A = R <= NPT;
    constexpr int NH = HOLD_A ? R : NPT, NS = HOLD_A ? NPT : R;
    auto compute = [&](int slot, int off, auto load, auto convert) {
        auto rd_a = [&](int r, int t) { return frag(fa0 + slot + split_a_plane(T, t, r * RPT, 0)); };
        auto rd_b = [&](int n, int t) {
            return frag(fb0[n] + off + split_x_plane(T, t, 0));
        };
        b8 H[NH][3], F[2][3];
#pragma unroll
        for (int t = 2; t >= 0; --t) {
#pragma unroll
            for (int h = 0; h < NH; ++h) H[h][t] = HOLD_A ? rd_a(h, t) : rd_b(h, t);
            F[0][2 - t] = HOLD_A ? rd_b(0, 2 - t) : rd_a(0, 2 - t);
        }
        __builtin_amdgcn_sched_barrier(0);
        load();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < NS; ++n) {
            constexpr int NM = 6 * NH;
            if (n + 1 < NS) {
#pragma unroll
                for (int t = 0; t < 3; ++t)
                    F[(n + 1) & 1][t] = HOLD_A ? rd_b(n + 1, t) : rd_a(n + 1, t);
            }
            if (n == NS - 2) convert(0);
            if (n == NS - 1) convert(1);
#pragma unroll
            for (int q = 0; q < 6; ++q)
#pragma unroll
                for (int h = 0; h < NH; ++h) {
                    if constexpr (HOLD_A)
                        acc[h][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            H[h][PA[q]], F[n & 1][PB[q]], acc[h][n], 0, 0, 0);
                    else
                        acc[n][h] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            F[n & 1][PB[q]], H[h][PA[q]], acc[n][h], 0, 0, 0);
                }
            const int nrd = n + 1 < NS ? 3 : 0;
#pragma unroll
            for (int i = 0; i < NM; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if (i < nrd) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                else if (n >= NS - 2) __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // Strips past the LP positions of a buffer are loaded but not kept.
    auto x_on = [&](int j) {
        constexpr int PER = T.waves() / T.nchi() * 64;
        return (j + 1) * PER <= LP || split_x_t(T, wave, lane, j) < LP;
    };
    float ra[CHI][NB], rx[CHI][NB];

    // Filters of the first step, input of the first stage.
    constexpr int AB = T.a_bytes(), XB = T.x_bytes();
    const int df = DF > 0 ? DF : a.df;
    const int n_stage = a.n_step / df;
    Pos cur{0, 0};
    load_a(0, ra);
    {
        const XDesc d = x_desc(cur);
#pragma unroll
        for (int j = 0; j < NXMAX; ++j)
            if (j < a.nx) {
                load_x(d, xgoff[j], rx);
                store_x(0, xlds[j], x_on(j), rx);
            }
    }
    store_a(0, ra);
    __syncthreads();

    int slot = 0;
    for (int st = 0; st < n_stage; ++st) {
        // (behind the last step, its filters and input are loaded again and
        // written where nothing reads them)
        const Pos nst = next_stage(cur);
        const XDesc xd = x_desc(nst);
        const int xb = (st & 1) * XB, xn = XB - xb;
        const int w_cur = cur.ci0 * a_chan + cur.rt * df * (NB * 4);
        const int w_nxt = nst.ci0 * a_chan + nst.rt * df * (NB * 4);
        auto step = [&](int qx) {
            const int wo = qx + 1 < df ? w_cur + (qx + 1) * (NB * 4) : w_nxt;
            if constexpr (DF > 0) {
                compute(slot, xb + qx * 16,
                        [&]() {
                            load_a(wo, ra);
                            load_x(xd, xgoff[qx], rx);
                        },
                        [&](int half) {
                            if (half == 0) store_a(AB - slot, ra);
                            else store_x(xn, xlds[qx], x_on(qx), rx);
                        });
            } else {
                // strip rounds qx xi ... of the next stage, the first of them
                // loaded with the filters
                compute(slot, xb + qx * 16,
                        [&]() {
                            load_a(wo, ra);
#pragma unroll
                            for (int j = 0; j < NXMAX; ++j)
                                if (j == qx * a.xi && j < a.nx) load_x(xd, xgoff[j], rx);
                        },
                        [&](int half) {
                            if (half == 1) store_a(AB - slot, ra);
                        });
#pragma unroll
                for (int j = 0; j < NXMAX; ++j)
                    if (j >= qx * a.xi && j < (qx + 1) * a.xi && j < a.nx) {
                        if (j > qx * a.xi) load_x(xd, xgoff[j], rx);
                        store_x(xn, xlds[j], x_on(j), rx);
                    }
            }
            __syncthreads();
            slot = AB - slot;
        };
        if constexpr (DF > 0) {
#pragma unroll
            for (int qx = 0; qx < DF; ++qx) step(qx);
        } else {
            for (int qx = 0; qx < df; ++qx) step(qx);
        }
        cur = nst;
    }

    // Infinite or NaN sums (of infinities, operands from 2^112, sums from 2^96): every row of a multivector is in this wave, so a filter blade
    // dropped with its zero sign shows in the row where its sign is not zero.
    float z = 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int n = 0; n < NPT; ++n)
#pragma unroll
            for (int e = 0; e < 16; ++e) z = fmaf(acc[r][n][e], 0.f, z);
    float unscale = SPLIT_UNSCALE;
    if (__ballot(z != 0.f)) {
        split_fp32_sums<KD, NB>(T, a, g, wave, lane, acc);
        unscale = 1.f;
    }

    // Epilogue: bias, optional activation; one lane holds a whole multivector.
    const bool has_act = a.act.mode >= 0;
    int gslot[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) gslot[i] = has_act ? gate_slot(a.act, i) : -1;
    const FastDiv fnpos = fast_div(a.npos);
    // element e of row r: with 16 channels to a row, odd rows are the row
    // tile's upper half
    auto el = [&](int r, int n, int e) { return acc[r / RPT][n][e + r % RPT * (CW / 2)]; };
#pragma unroll
    for (int np = 0; np < NPT; ++np) {
        const int m = split_out_m(T, g, wave, lane, np);
#pragma unroll
        for (int e = 0; e < CW / 2; ++e) {
            const int co = split_out_co(T, g, wave, lane, e);
            if (m >= g.m_end || co >= a.C_out) continue;
            float v[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) v[blade_perm(NB, i)] = el(i, np, e) * unscale;
            if (a.bias) {
#pragma unroll
                for (int i = 0; i < NB; ++i) v[i] += a.bias[co * NB + i];
            }
            if (has_act) {
                float part = 0.f;
#pragma unroll
                for (int i = 0; i < NB; ++i) part += gate_coef(a.act, gslot[i], co) * v[i];
                const float gate = gate_sigmoid(a.act, part, co);
#pragma unroll
                for (int i = 0; i < NB; ++i) v[i] *= gate;
            }
            float* const yp = a.y + split_out_ofs(a, fnpos, m, co) * NB;
            if constexpr (NB == 2) {
                *reinterpret_cast<f2*>(yp) = f2{v[0], v[1]};
            } else {
#pragma unroll
                for (int h = 0; h < NB / 4; ++h)
                    reinterpret_cast<f4*>(yp)[h] =
                        f4{v[4 * h], v[4 * h + 1], v[4 * h + 2], v[4 * h + 3]};
            }
        }
    }
}

template <int KD, int NB, int DF, int WCO, int WPOS, int NPT, int LP, int CW>
cliff_status run(const ConvProblem& p, hipStream_t stream, int64_t* blocks)
{
    constexpr SplitTile T{KD, NB, WCO, WPOS, NPT, LP, CW};
    static_assert(T.lds_bytes() <= 160 * 1024, "LDS");
    const int64_t D = p.d_image, Do = p.d_out, df = p.d_filter, P = T.pos();
    int64_t npos = 1, img = 1, taps = 1;
    for (int t = 0; t < KD; ++t) {
        npos *= Do;
        img *= D;
        taps *= df;
    }
    const int64_t M = p.B * npos;
    // 32-bit position indices; input offsets are 32-bit multivector counts
    // from the block's first row, which spans at most `rows` output rows
    const int64_t cross = (P - 1 + Do - 1) / Do, rows = cross + 1;
    const int64_t entries = KD == 1 ? rows : rows / (npos / Do) + 2;
    // and, like those of the filters, 31-bit byte offsets
    if (M >= (1ll << 31) - P || (entries + 1) * p.C_in * img * NB * 4 >= (1ll << 31) ||
        (p.C_in + T.cpg()) * p.C_out * taps * NB * 4 >= (1ll << 31))
        return CLIFF_EUNSUPPORTED;
    // the longest run of input positions of a block
    const int64_t L = P + (cross + 1) * (df - 1);
    constexpr int per_round = T.waves() / T.nchi() * 64;
    const int64_t nx = (L + per_round - 1) / per_round;
    const int64_t xi = (nx + df - 1) / df;
    if (L > LP || nx > split_rounds(KD, DF) || xi > (DF > 0 ? 1 : 2)) return CLIFF_EUNSUPPORTED;
    const int64_t n_co_blk = (p.C_out + T.co_wg() - 1) / T.co_wg();
    const int64_t n_blk = (M + P - 1) / P * n_co_blk;
    const int64_t n_grp = (p.C_in + T.cpg() - 1) / T.cpg();
    if (n_blk >= (1ll << 31) || n_grp * taps >= (1ll << 31)) return CLIFF_EUNSUPPORTED;
    if (blocks) {  // a plan only
        *blocks = n_blk;
        return CLIFF_OK;
    }

    SplitArgs a;
    a.x = p.x;
    a.w = p.w;
    a.bias = p.bias;
    a.y = p.y;
    a.C_in = (int)p.C_in;
    a.C_out = (int)p.C_out;
    a.D = (int)D;
    a.Do = (int)Do;
    a.df = (int)df;
    a.M = (int)M;
    a.npos = (int)npos;
    a.nrow = (int)(M / Do);
    a.taps = (int)taps;
    a.nrt = (int)(taps / df);
    a.n_step = (int)(n_grp * taps);
    a.n_co_blk = (int)n_co_blk;
    a.n_blk = (int)n_blk;
    a.nx = (int)nx;
    a.xi = (int)xi;
    a.cin_stride = (int)img;
    a.sign = p.sign;
    a.act = p.act;
    for (int i = 0; i < NB; ++i)
        for (int h = 0; h < NB / 2; ++h) {
            uint32_t sx = 0, sz = 0;
            for (int e = 0; e < 2; ++e) {
                const float s = sign_of(p.sign, blade_perm(NB, i) * NB + blade_perm(NB, 2 * h + e));
                sx |= (s < 0.f ? 0x8000u : 0u) << (16 * e);
                sz |= (s != 0.f ? 0xffffu : 0u) << (16 * e);
            }
            a.sx[i * (NB / 2) + h] = sx;
            a.sz[i * (NB / 2) + h] = sz;
        }
    if (debug_enabled())
        fprintf(stderr,
                "cliffconv: conv_split k=%d d_filter=%d, %d channels x %d positions, "
                "%lld workgroups of %d, %d LDS bytes\n",
                KD, (int)df, T.co_wg(), (int)P, (long long)n_blk,
                T.nt(), T.lds_bytes());
    if (observe_launch(LAUNCH_CONV_SPLIT, {KD, NB, DF, WCO, WPOS, NPT, LP, CW}, n_blk, T.nt(),
                       T.lds_bytes(), &a))
        return CLIFF_OK;
    clear_hip_error();
    hipLaunchKernelGGL((conv_split_kernel<KD, NB, DF, WCO, WPOS, NPT, LP, CW>), dim3((unsigned)n_blk),
                       dim3(T.nt()), (size_t)T.lds_bytes(), stream, a);
    return hipGetLastError() == hipSuccess ? CLIFF_OK : CLIFF_EDEVICE;
}

// One tile shape: its launcher (or planner), and the microseconds of one step
// (one K group of one tap, at 3 taps a row) with one and with two workgroups
// on every CU, measured on MI355X at 256 and 512 workgroups (8-wave workgroups
// fill a CU alone).
struct Shape {
    cliff_status (*run)(const ConvProblem&, hipStream_t, int64_t*);
    int cpg, cw;
    double t1, t2;
};
template <int KD, int NB, int DF, int WCO, int WPOS, int NPT, int LP, int CW = 32>
constexpr Shape shape(double t1, double t2)
{
    return Shape{run<KD, NB, DF, WCO, WPOS, NPT, LP, CW>,
                 SplitTile{KD, NB, WCO, WPOS, NPT, LP, CW}.cpg(), CW, t1, t2};
}

template <int DF>
cliff_status launch_df(const ConvProblem& p, hipStream_t stream, double most_us)
{
    // k = 1, channels x positions: 64 x 256, 64 x 128, 64 x 512, 32 x 512, 32 x 256
    static constexpr Shape shapes1[] = {
        shape<1, 2, 0, 2, 4, 2, 512>(1.70, 3.40), shape<1, 2, 0, 2, 2, 2, 256>(1.08, 1.76),
        shape<1, 2, 0, 2, 4, 4, 724>(3.10, 6.20), shape<1, 2, 0, 1, 8, 2, 724>(1.78, 3.56),
        shape<1, 2, 0, 1, 4, 2, 360>(1.10, 1.83)};
    // k = 2: 64 x 256, 64 x 128, 32 x 256, 32 x 128, 64 x 64, 16 x 256 (16 x 128
    // never ahead: 62 against 59, 217 against 193 us)
    static constexpr Shape shapes2[] = {
        shape<2, 4, DF, 2, 4, 2, 320>(2.13, 4.18), shape<2, 4, DF, 2, 2, 2, 168>(1.19, 2.23),
        shape<2, 4, DF, 1, 8, 1, 320>(1.12, 2.20), shape<2, 4, DF, 1, 4, 1, 168>(0.76, 1.27),
        shape<2, 4, DF, 2, 2, 1, 100>(0.75, 1.36),
        shape<2, 4, DF, 1, 8, 1, 320, 16>(0.75, 1.25)};
    // k = 3: 32 x 128, 32 x 256
    static constexpr Shape shapes3[] = {shape<3, 8, DF, 1, 4, 1, 168>(1.48, 2.28),
                                        shape<3, 8, DF, 1, 8, 1, 320>(2.10, 4.17)};
    const Shape* const s = p.k == 1 ? shapes1 : p.k == 2 ? shapes2 : shapes3;
    const int n = p.k == 1 ? 5 : p.k == 2 ? 6 : 2;
    const int cus = device_cus();
    if (cus < 1) return CLIFF_EUNSUPPORTED;
    // Estimate: the CU with the most workgroups takes them in pairs; a step
    // with `df` taps a row converts 1 / df of a stage's input (fitted at 3 and
    // 5 taps); 5 us of launch, prologue and epilogue.
    const double df = (double)p.d_filter;
    const Shape* best = nullptr;
    double best_us = most_us;
    for (int i = 0; i < n; ++i) {
        int64_t blocks = 0;
        // 16 channels only where blocks of 32 leave half of the last one empty
        // (others were not measured)
        if (s[i].cw == 16 && (p.C_out - 1) % 32 >= 16) continue;
        if (s[i].run(p, stream, &blocks) != CLIFF_OK) continue;
        const int64_t w = (blocks + cus - 1) / cus;
        const double steps = (double)((p.C_in + s[i].cpg - 1) / s[i].cpg) * std::pow(df, p.k);
        const double us = 5.0 + steps * (0.67 + 1.0 / df) *
                                    ((double)(w / 2) * s[i].t2 + (double)(w % 2) * s[i].t1);
        if (us < best_us) {
            best_us = us;
            best = &s[i];
        }
    }
    return best ? best->run(p, stream, nullptr) : CLIFF_EUNSUPPORTED;
}

}  // namespace

cliff_status launch_conv_split(const ConvProblem& p, hipStream_t stream)
{
    if (launch_observer && launch_observer->last_kind < LAUNCH_CONV_SPLIT) return CLIFF_EUNSUPPORTED;
    if (p.d_filter < 2) return CLIFF_EUNSUPPORTED;
    // A sum's error goes with its roundings: a tap costs six here for every 8 K
    // slots in use (the error steps with 8, not with an MFMA's 16), and one on the
    // fp32 tiles for every product that the table does not make zero.  Tables
    // without zeros: 0.80 to 0.97 of the fp32 tiles' error (2-norm, all C_in and
    // filters, up to 18816 products).  With zeros it is 0.87 to 0.995 while there are
    // at most 1.1 times as many roundings (k = 3 tables of one zero; k = 2 with even
    // C_in or C_in >= 11).  Past that it grows with the products of a sum: C_in 7 and
    // 9 at k = 2 0.98 at 189 products, 1.00 at 525, 1.007 at 1029; k = 3 with two
    // zeros 0.995 at 576, 1.05 at 7776; C_in 3 and 5 at k = 2 0.99 to 1.05.
    if (p.sign.zero) {
        const int64_t cpc = 8 / p.nb, nz = p.nb * p.nb - __builtin_popcountll(p.sign.zero);
        const double products = (double)p.C_in * nz / p.nb;  // of a tap
        if (6.0 * (double)((p.C_in + cpc - 1) / cpc) > 1.1 * products &&
            ((p.k == 2 && p.C_in < 7) || products * std::pow((double)p.d_filter, p.k) > 500.0))
            return CLIFF_EUNSUPPORTED;
    }
    // One K group with padding channels at four taps or less: the output's stores
    // are most of the time and hidden by too little (k = 2, 2x2 filters, C_in 3,
    // 62 channels, B 13, d 324 491 us on the fp32 tiles, 544 here; C_in 4, 63
    // channels, B 5, d 488 516, 465).
    if (p.C_in < 16 / p.nb && std::pow((double)p.d_filter, p.k) <= 4) return CLIFF_EUNSUPPORTED;
    // Taken where the estimate is below the time of the fp32 tiles at their
    // best rate (146 TFLOP/s, 0.93 of the fp32 peak, on the largest layers;
    // 141 for k = 1); smaller layers, where that rate is out of reach for
    // either, stay there.
    double useful = 2.0 * (double)p.B * p.C_out * p.C_in * p.nb * p.nb;
    for (int t = 0; t < p.k; ++t) useful *= (double)p.d_out * p.d_filter;
    const double most_us = useful / (p.k == 1 ? 141e6 : 146e6);
    return p.k > 1 && p.d_filter == 3 ? launch_df<3>(p, stream, most_us) : launch_df<0>(p, stream, most_us);
}

}  // namespace cliff
