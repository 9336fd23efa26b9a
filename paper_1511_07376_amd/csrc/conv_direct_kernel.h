// Convolution for layers with few output tiles, without staging.
//
// A wave owns FM x FN blocks of 32 output channels x 32 output pixels and
// feeds the fp32 matrix cores from its own registers: lane (i, h) loads taps
// 8h .. 8h + 7 of a 16-tap run of its channel's weights and of its pixel's
// window (half h is the k index of v_mfma_f32_32x32x2_f32; any order of the
// taps will do).  The KW waves of a workgroup take the runs in turn and their
// partial tiles are summed through LDS in wave order.  So a layer whose whole
// output is a hundred tiles runs on several waves per SIMD in one launch, with
// no barrier in the reduction loop and no atomics, where the tiled kernels
// need a bias fill, a split reduction and a ReLU pass.  (Layers of at most 64
// tiles and long reductions are split here as well.)
//
// What bounds it is the latency of a run's loads (few runs a wave) and then
// the texture addresser: a block's operands are loaded by every wave that
// needs them, so large outputs stay with the tiled kernels.  Splitting the
// operands into bf16 parts here costs as many vector instructions per block
// as the fp32 matrix instructions take cycles, and measured the same.
// 20x12x12 -> 50, 5x5, 16 images: 18.5 -> 7.2 us; 64x56x56 -> 64, 3x3, one
// image: 19.9 -> 8.2 us; AlexNet's conv2 on one image: 21.1 -> 12.3 us (times
// of a call, fill and ReLU pass included).
#pragma once

#include "conv_igemm_kernel.h"

namespace cnn {
namespace conv {

template <int FM, int FN, int KW, bool VEC_W, int WINDOW>
__global__ void __launch_bounds__(64 * KW)
conv2d_direct_f32(ConvParams p) {
    constexpr int TM = FM * 32, TN = FN * 32, NT = 64 * KW, TILES = FM * FN;
    constexpr int D = kDirectStages;  // runs of loads in flight
    extern __shared__ __attribute__((aligned(16))) int stab[];
    __shared__ float red[KW * TILES * 1024];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int g = blockIdx.z % p.G;
    const int kbeg = (blockIdx.z / p.G) * p.kchunk;
    const int klen = min(p.kchunk, p.Kr - kbeg);
    int m0, k0;
    {
        const int gy = gridDim.y, tiles = gridDim.x * gy;
        const int wg = blockIdx.x + gridDim.x * blockIdx.y;
        const int full = tiles & ~7;
        const int seq = wg < full ? (wg & 7) * (full >> 3) + (wg >> 3) : wg;
        m0 = (seq / gy) * TN;
        k0 = (seq % gy) * TM;
    }
    // tap table, padded to a whole round of runs plus the runs in flight
    const int nrun = (klen + 15) / 16;
    const int niter = (nrun + KW - 1) / KW;  // runs per wave
    const int ntab = direct_table_entries(p.kchunk, KW);
    for (int kk = threadIdx.x; kk < ntab; kk += NT) {
        const int c = (int)fdiv(kbeg + kk, p.f_rs);
        const int rs = kbeg + kk - c * p.RS;
        const int r = (int)fdiv(rs, p.f_s);
        const int s = rs - r * p.S;
        const int toff = ((c * p.H + r) * p.W + s) * 4;
        const bool in = kk < klen;
        if constexpr (WINDOW == kWindowNoPad) {
            stab[kk] = in ? toff : kOutOfRange;
        } else if constexpr (WINDOW == kWindowMask) {
            stab[kk] = in ? (toff << 5) | rs : 31;
        } else {
            stab[kk] = toff;
            stab[ntab + kk] = in ? (r << 16) | s : 0x7fff0000;
        }
    }
    // this lane's pixels
    int hb[FN], wb[FN], pix[FN];
    unsigned inv[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        const int m = m0 + j * 32 + l32;
        const int mc = min(m, p.M - 1);
        const int n = (int)fdiv(mc, p.f_pq);
        const int pq = mc - n * p.PQ;
        const int pp = (int)fdiv(pq, p.f_q);
        hb[j] = pp * p.sh - p.ph;
        wb[j] = (pq - pp * p.Q) * p.sw - p.pw;
        pix[j] = ((n * p.C + g * p.Cg) * p.HW + hb[j] * p.W + wb[j]) * 4;
        if constexpr (WINDOW == kWindowMask)
            inv[j] = 0x80000000u | outside_taps<unsigned>(hb[j], wb[j], p.H, p.W, p.R, p.S);
    }
    const __amdgpu_buffer_rsrc_t xres =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.x), (short)0, p.xbytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t wres =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.w), (short)0, p.wbytes, 0x00020000);
    int wrow[FM];
    bool wok[FM];
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        wok[i] = k0 + i * 32 + l32 < p.Kg;
        wrow[i] = ((g * p.Kg + min(k0 + i * 32 + l32, p.Kg - 1)) * p.Kr + kbeg + half * 8) * 4;
    }
    __syncthreads();

    float xr[D][FN][8], wr[D][FM][8];
    auto load = [&](int run, int sg) __attribute__((always_inline)) {
        const int k = run * 16 + half * 8;  // this lane's first tap of the run
#pragma unroll
        for (int u0 = 0; u0 < 8; u0 += 4) {
            const int4 e4 = *reinterpret_cast<const int4*>(&stab[k + u0]);
            const int e[4] = {e4.x, e4.y, e4.z, e4.w};
            int4 f4;
            if constexpr (WINDOW == kWindowAny) f4 = *reinterpret_cast<const int4*>(&stab[ntab + k + u0]);
            const int rs[4] = {f4.x, f4.y, f4.z, f4.w};
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    int voff;
                    if constexpr (WINDOW == kWindowNoPad) {
                        voff = (int)((unsigned)pix[j] + (unsigned)e[u]);
                    } else if constexpr (WINDOW == kWindowMask) {
                        voff = (pix[j] + (int)((unsigned)e[u] >> 5)) | (int)(((inv[j] >> (e[u] & 31)) & 1u) << 31);
                    } else {
                        const bool in = (unsigned)(hb[j] + (rs[u] >> 16)) < (unsigned)p.H &&
                                        (unsigned)(wb[j] + (rs[u] & 0xffff)) < (unsigned)p.W;
                        voff = in ? pix[j] + e[u] : kOutOfRange;
                    }
                    xr[sg][j][u0 + u] =
                        __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xres, voff, 0, 0));
                }
        }
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            if constexpr (VEC_W) {
#pragma unroll
                for (int u = 0; u < 8; u += 4) {
                    typedef float f32x4 __attribute__((ext_vector_type(4)));
                    const int voff = wok[i] && k + u < klen ? wrow[i] + (run * 16 + u) * 4 : kOutOfRange;
                    const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(wres, voff, 0, 0));
#pragma unroll
                    for (int q = 0; q < 4; ++q) wr[sg][i][u + q] = v[q];
                }
            } else {
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int voff = wok[i] && k + u < klen ? wrow[i] + (run * 16 + u) * 4 : kOutOfRange;
                    wr[sg][i][u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wres, voff, 0, 0));
                }
            }
        }
    };
    floatx16 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
    auto compute = [&](int sg) __attribute__((always_inline)) {
        if (p.relu_x) {  // uniform
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int u = 0; u < 8; ++u) xr[sg][j][u] = xr[sg][j][u] > 0.0f ? xr[sg][j][u] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(wr[sg][i][u], xr[sg][j][u], acc[i][j], 0, 0, 0);
    };
    // runs wave, wave + KW, ...; past the chunk the table and the weights read as zero
#pragma unroll
    for (int d = 0; d < D; ++d) load(d * KW + wave, d);
    for (int it = 0; it < niter; it += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (it + d < niter) compute(d);  // uniform
            if (it + d + D < niter) load((it + d + D) * KW + wave, d);
        }
    }

    // ---- the waves' partial tiles, summed in wave order
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                red[((wave * TILES + i * FN + j) * 16 + v) * 64 + lane] = acc[i][j][v];
    __syncthreads();
    for (int e = threadIdx.x; e < TILES * 1024; e += NT) {
        float sum = red[e];
#pragma unroll
        for (int w = 1; w < KW; ++w) sum += red[w * TILES * 1024 + e];
        const int t = e >> 10, v = (e >> 6) & 15, l = e & 63;
        const int kr = k0 + (t / FN) * 32 + 8 * (v >> 2) + 4 * (l >> 5) + (v & 3);
        const int m = m0 + (t % FN) * 32 + (l & 31);
        if (kr >= p.Kg || m >= p.M) continue;
        const int n = (int)fdiv(m, p.f_pq), pq = m - n * p.PQ;
        const int ko = g * p.Kg + kr;
        float* dst = p.y + (n * p.K + ko) * p.PQ + pq;
        if (p.splits > 1) {
            atomicAdd(dst, sum);
        } else {
            if (p.bias) sum += p.bias[ko];
            if (p.relu) sum = sum > 0.0f ? sum : 0.0f;
            *dst = sum;
        }
    }
}

}  // namespace conv
}  // namespace cnn
