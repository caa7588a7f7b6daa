// Clifford linear layer (paper, Algorithm 2) for large batches on the bf16
// matrix cores with fp32 accuracy: Y = X E^T + bias with E the expanded
// weight, every operand split into the three bf16 parts of split.hpp and every
// product into six, summed in fp32 by v_mfma_f32_32x32x16_bf16.
//
// Bound by HBM: at 32 FLOP per byte (128 columns in and out) the fp32 matrix
// cores need as long as the memory, and the two together took 1.4 times the
// memory's time; six bf16 products take half of it and overlap.
//
// Every workgroup (8 waves, one per CU) expands and splits the weight into LDS
// once ([part][chunk of 8 K slots][column], read as fragments without
// conflicts), then each wave streams tiles of 32 rows of X with no barrier:
// the rows go from HBM straight into registers in fragment order, PF groups of
// 16 K values ahead and across tiles, and are split there; one tile's stores
// and the next one's loads drain under the MFMAs.
//
// Measured against the fp32 kernel (linear_mfma.hip), g = (1, 1): 32 -> 32
// channels, B = 2^20 297 -> 242 us (4.4 TB/s; a device copy of the same bytes
// runs at 5.3), 2^18 81 -> 54, 2^16 29 -> 19.4 us; 64 -> 16, 2^20 308 -> 278;
// 16 -> 32, 2^20 188 -> 187; 32 -> 16 185 -> 166; error against 64 bits 0.75 to
// 0.98 times (signatures with two zeros) the fp32 kernel's.  Loads and stores of 64
// contiguous bytes of 16 rows, with an exchange of lane rows behind them,
// instead of 32 bytes of 32 rows: 277 -> 238 us.  8 groups of prefetch instead
// of 4: 242.  64 -> 256 columns spill (8 row tiles) and stay there, as do
// 64 -> 64, at the memory's rate already, and 256 -> 256.
//
// Tiles with a result that is not finite (infinities, operands from 2^112 and sums
// from 2^96 on) are computed again on the fp32 matrix cores after the wave's last
// one: with a channel of the lowest value in all rows but 32, 2^17 rows of 32 -> 32
// channels take 91 us instead of 36 (fp32 kernel 64; half of 2^18 rows masked and
// one lane for an output: 437).
#include <stdio.h>

#include <algorithm>

#include "common.hpp"
#include "epilogue.hpp"
#include "linear_split_geom.hpp"
#include "split.hpp"

namespace cliff {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f16 __attribute__((ext_vector_type(16)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

// Lane rows (16 lanes) 1 and 3 of a change places with lane rows 0 and 2 of b.
__device__ inline void exchange(f4& a, f4& b)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float x = a[e], y = b[e];
        const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, x),
                                                        __builtin_bit_cast(uint32_t, y), false, false);
        const uint32_t r0 = r[0], r1 = r[1];
        a[e] = __builtin_bit_cast(float, r0);
        b[e] = __builtin_bit_cast(float, r1);
    }
}

template <int NB, int RT, int KQ, int PF>
__global__ __launch_bounds__(512, 2) void linear_split_kernel(LinSplitArgs a)
{
    static_assert(KQ % PF == 0, "whole prefetch rounds per tile");
    constexpr LinSplitShape S{NB, RT, KQ};
    constexpr int N = S.N(), K = S.K(), PL = S.plane(), CO = N / NB;
    extern __shared__ u4 smem4[];
    char* const wl = reinterpret_cast<char*>(smem4);
    float* const bl = reinterpret_cast<float*>(wl + S.tail());
    float* const cl = bl + N;
    float* const gl = cl + N;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    for (int e = tid; e < S.items(); e += 512) {
        const int co = lsp_w_co(S, e), chunk = lsp_w_chunk(S, e);
        float w[8];  // blades of the chunk's input channels
#pragma unroll
        for (int u = 0; u < 8; ++u)
            w[u] = a.w[lsp_w_float(S, (8 * chunk + u) / NB, co) + u % NB];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            Parts p[4];
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                float v[2];
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const int u = 2 * h + c, j = u % NB;
                    v[c] = sign_of(a.sign, i * NB + j) * w[u / NB * NB + src_blade(NB, i, j)];
                }
                p[h] = split2(v[0], v[1]);
            }
#pragma unroll
            for (int t = 0; t < 3; ++t)
                *reinterpret_cast<u4*>(wl + t * PL + lsp_a_byte(S, chunk, co * NB + i)) =
                    u4{p[0].t[t], p[1].t[t], p[2].t[t], p[3].t[t]};
        }
    }
    for (int e = tid; e < N; e += 512) {
        bl[e] = a.bias ? a.bias[e] : 0.f;
        cl[e] = a.act.mode >= 0 ? gate_coef(a.act, gate_slot(a.act, e % NB), e / NB) : 0.f;
        if (e < CO) gl[e] = a.act.mode == CLIFF_AGG_LINEAR ? a.act.bias[e] : 0.f;
    }
    __syncthreads();

    const int64_t stride = (int64_t)gridDim.x * 8;
    const int64_t t0 = (int64_t)blockIdx.x * 8 + wave;
    if (t0 >= a.n_tile) return;  // wave-uniform, after the only barrier
    // Rows past B lie past the descriptor's end: loads give zeros, stores
    // nothing.
    auto x_desc = [&](int64_t t) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.x) + 32 * t * K, (short)0,
                                                 lsp_rows(a, t) * K * 4, 0x00020000);
    };
    const int xo = lsp_x_float(S, lane, 0, 0) * 4;
    constexpr int xh = (lsp_x_float(S, 0, 0, 1) - lsp_x_float(S, 0, 0, 0)) * 4;
    f4 ring[PF][2];
    auto load = [&](__amdgpu_buffer_rsrc_t d, int s, f4 (&v)[2]) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            v[h] = __builtin_bit_cast(
                f4, __builtin_amdgcn_raw_buffer_load_b128(d, xo + xh * h + 64 * s, 0, 0));
    };
    const char* const fa = wl + lsp_a_byte(S, lane >> 5, lane & 31);
    f16 acc[RT];
    constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
    // the parts of a K group's values of this lane's row
    auto split_group = [&](const f4 (&w)[2], u4 (&b)[3]) {
        f4 v[2] = {w[0], w[1]};
        exchange(v[0], v[1]);
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const Parts p = split2(v[h >> 1][2 * (h & 1)], v[h >> 1][2 * (h & 1) + 1]);
#pragma unroll
            for (int q = 0; q < 3; ++q) b[q][h] = p.t[q];
        }
    };
    auto read_a = [&](int s, int r, b8 (&A)[3]) {
#pragma unroll
        for (int q = 0; q < 3; ++q)
            A[q] = *reinterpret_cast<const b8*>(fa + q * PL + lsp_a_byte(S, 2 * s, 32 * r));
    };
    // One tile's K loop, unrolled; the prefetch runs on into tile tn.  The
    // fragments of the next row tile are read, and the next K group's values
    // split, between the MFMAs of this one.
    auto tile = [&](int64_t t, int64_t tn) {
        const __amdgpu_buffer_rsrc_t dc = x_desc(t), dn = x_desc(tn);
        b8 A[2][3];
        u4 b[2][3];
        split_group(ring[0], b[0]);
        read_a(0, 0, A[0]);
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[r][e] = 0.f;
#pragma unroll
        for (int s = 0; s < KQ; ++s) {
            // (slot s % PF was split in the step before)
            if (s + PF < KQ) load(dc, s + PF, ring[s % PF]);
            else load(dn, s + PF - KQ, ring[s % PF]);
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                const int cur = (s * RT + r) & 1;
                if (r + 1 < RT) read_a(s, r + 1, A[cur ^ 1]);
                else if (s + 1 < KQ) read_a(s + 1, 0, A[cur ^ 1]);
                if (r == RT - 1 && s + 1 < KQ) split_group(ring[(s + 1) % PF], b[(s + 1) & 1]);
#pragma unroll
                for (int q = 0; q < 6; ++q)
                    acc[r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        A[cur][PA[q]], __builtin_bit_cast(b8, b[s & 1][PB[q]]), acc[r], 0, 0, 0);
#pragma unroll
                for (int q = 0; q < 6; ++q) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    if (q < 3) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    if (r == RT - 1) __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    const bool has_act = a.act.mode >= 0;
    const bool mean = a.act.mode == CLIFF_AGG_MEAN;
    auto gate = [&](float sum, const float* bias, int co) {
        float s = sum + bias[co];
        if (mean) s = s / (float)a.act.K;
        return 1.0f / (1.0f + __expf(-s));
    };
    // Tile t's outputs from the accumulators, which hold 1 / unscale times its
    // sums; whether one of them is infinite or NaN (in any lane).
    auto finish = [&](int64_t t, float unscale) {
        float z = 0.f;
        const __amdgpu_buffer_rsrc_t yd = __builtin_amdgcn_make_buffer_rsrc(
            a.y + 32 * t * N, (short)0, lsp_rows(a, t) * N * 4, 0x00020000);
        // the bias and gate parameters are the same for every tile; an opaque
        // zero keeps their LDS reads here instead of in registers
        int opq = 0;
        __asm__ volatile("" : "+s"(opq));
        const float* const ble = bl + opq;
        const float* const cle = cl + opq;
        const float* const gle = gl + opq;
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                f4 o[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int q = 2 * u + h, n = lsp_y_col(S, lane, r, q);
                    const f4 bb = *reinterpret_cast<const f4*>(ble + n);
                    f4& v = o[h];
                    v = f4{acc[r][4 * q], acc[r][4 * q + 1], acc[r][4 * q + 2], acc[r][4 * q + 3]} * unscale +
                        bb;
                    if (has_act) {
                        const f4 cf = *reinterpret_cast<const f4*>(cle + n);
                        if constexpr (NB == 2) {
                            const float g0 = gate(cf[0] * v[0] + cf[1] * v[1], gle, n / 2);
                            const float g1 = gate(cf[2] * v[2] + cf[3] * v[3], gle, n / 2 + 1);
                            v[0] *= g0;
                            v[1] *= g0;
                            v[2] *= g1;
                            v[3] *= g1;
                        } else {
                            float part = cf[0] * v[0] + cf[1] * v[1] + cf[2] * v[2] + cf[3] * v[3];
                            // N_B = 8: the other half of the multivector is in lane ^ 32
                            if (NB == 8) part += __shfl_xor(part, 32);
                            v *= gate(part, gle, n / NB);
                        }
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) z = fmaf(v[e], 0.f, z);
                }
                exchange(o[0], o[1]);
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, o[h]), yd,
                                                           lsp_y_float(S, lane, r, u, h) * 4, 0, 0);
            }
        return __ballot(z != 0.f) != 0;
    };
    {
        const __amdgpu_buffer_rsrc_t d = x_desc(t0);
#pragma unroll
        for (int p = 0; p < PF; ++p) load(d, p, ring[p]);
    }
    uint64_t bad = 0;  // bit i % 64: the wave's tile i has an infinite or NaN output
    int i = 0;
    int64_t t = t0, tn = t + stride;
    tile(t, tn < a.n_tile ? tn : t);
    for (;; ++i) {
        bad |= (uint64_t)finish(t, SPLIT_UNSCALE) << (i & 63);
        if (tn >= a.n_tile) break;
        t = tn;
        tn = t + stride;
        tile(t, tn < a.n_tile ? tn : t);
    }
    if (bad == 0) return;
    // Those tiles (and any that share their bit) again as fp32 products on the
    // fp32 matrix cores, operands straight from memory, one input channel at a
    // time: values that bf16 parts cannot hold.
    i = 0;
    for (t = t0; t < a.n_tile; t += stride, ++i) {
        if (!(bad >> (i & 63) & 1)) continue;
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[r][e] = 0.f;
        for (int ci = 0; ci < a.C_in; ++ci)
#pragma unroll
            for (int h = 0; h < NB / 2; ++h) {
                const float xv = a.x[lsp_redo_x(S, a, t, lane, ci, h)];
                const int j = lsp_redo_j(S, lane, h);
#pragma unroll
                for (int r = 0; r < RT; ++r) {
                    const float wv = sign_of(a.sign, (lane & 31) % NB * NB + j) *
                                     a.w[lsp_redo_w(S, lane, r, ci, h)];
                    acc[r] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv, xv, acc[r], 0, 0, 0);
                }
            }
        finish(t, 1.f);
    }
}

template <int NB, int RT, int KQ>
cliff_status run(const ConvProblem& p, hipStream_t stream)
{
    constexpr int PF = KQ < 4 ? KQ : 4;
    constexpr LinSplitShape S{NB, RT, KQ};
    static_assert(S.lds_bytes() <= 160 * 1024, "LDS");
    LinSplitArgs a;
    a.x = p.x;
    a.w = p.w;
    a.bias = p.bias;
    a.y = p.y;
    a.B = p.B;
    a.n_tile = (p.B + 31) / 32;
    a.C_in = (int)p.C_in;
    a.C_out = (int)p.C_out;
    a.sign = p.sign;
    a.act = p.act;
    const int cus = device_cus();
    if (cus < 1) return CLIFF_EDEVICE;
    const int64_t n_wg = std::min<int64_t>((a.n_tile + 7) / 8, cus);
    if (debug_enabled())
        fprintf(stderr, "cliffconv: linear_split N_B=%d N=%d K=%d, %lld workgroups, %d LDS bytes\n", NB,
                S.N(), S.K(), (long long)n_wg, S.lds_bytes());
    if (observe_launch(LAUNCH_LINEAR_SPLIT, {NB, RT, KQ, PF}, n_wg, 512, S.lds_bytes(), &a))
        return CLIFF_OK;
    clear_hip_error();
    hipLaunchKernelGGL((linear_split_kernel<NB, RT, KQ, PF>), dim3((unsigned)n_wg), dim3(512),
                       (size_t)S.lds_bytes(), stream, a);
    return hipGetLastError() == hipSuccess ? CLIFF_OK : CLIFF_EDEVICE;
}

template <int NB>
cliff_status run_nk(const ConvProblem& p, hipStream_t stream)
{
    const int64_t n = p.C_out * NB, k = p.C_in * NB;
    if (n == 128 && k == 128) return run<NB, 4, 8>(p, stream);
    if (n == 128 && k == 64) return run<NB, 4, 4>(p, stream);
    if (n == 64 && k == 128) return run<NB, 2, 8>(p, stream);
    if (n == 64 && k == 256) return run<NB, 2, 16>(p, stream);
    return CLIFF_EUNSUPPORTED;
}

}  // namespace

cliff_status launch_linear_split(const ConvProblem& p, hipStream_t stream)
{
    if (launch_observer && launch_observer->last_kind < LAUNCH_LINEAR_SPLIT)
        return CLIFF_EUNSUPPORTED;
    if (p.d_image != 1 || p.d_filter != 1) return CLIFF_EUNSUPPORTED;
    // Rows from which it is ahead of the fp32 streamed kernel, which fills its
    // first round of waves at 32768 rows.  Every workgroup expands the weight first:
    // 128 columns of k = 3, and 64 -> 128, lose until then (32768 rows of 16 -> 16
    // channels, k = 3: 17.0 us, fp32 15.5; 40000: 17.3, 24.1; k = 2, 16 -> 32:
    // 12.5, 12.1; 40000: 12.4, 17.4), 128 -> 128 of k = 1 and 2 until about 18000
    // (k = 2: 16384 rows 14.9, 14.6; 20480: 15.0, 15.4); 64 columns are ahead
    // from 16384 on (k = 2, 128 -> 64: 11.6, 15.4).
    const bool wide = p.C_out * p.nb == 128;
    const int64_t rows = !wide ? 16384 : p.nb == 8 || p.C_in * p.nb == 64 ? 32769 : 18432;
    if (p.B < rows) return CLIFF_EUNSUPPORTED;
    switch (p.nb) {
        case 2: return run_nk<2>(p, stream);
        case 4: return run_nk<4>(p, stream);
        case 8: return run_nk<8>(p, stream);
    }
    return CLIFF_EUNSUPPORTED;
}

}  // namespace cliff
