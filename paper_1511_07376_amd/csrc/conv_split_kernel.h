// The im2col convolution of conv_igemm_kernel.h on the bf16 matrix cores.
//
// An fp32 value is the exact sum of three bf16 parts (bf16_split.h; 24
// significant bits in three times 8, each part's rounding error passed on to
// the next).  A product of two values is then nine products of parts, of which the three below 2^-24 of the whole are
// left out, and a v_mfma_f32_32x32x16_bf16 multiplies 16 taps in the time in
// which the fp32 matrix instruction multiplies one (32 against 64 cycles for
// 16 against 2 taps): six of them cost 3/8 of the fp32 time.
//
// Accuracy: the leading products are summed in one fp32 accumulator (one
// rounding per 16 taps) and the five smaller ones in a second, added at the
// end.  Against 64-bit sums the error is 0.3 to 0.9 of the fp32 matrix
// instruction's chain for 2 to 4608 taps of random values, signed or not
// (1200 taps: 0.4 to 0.8; a single tap: 1.02 to 1.03, for the products left
// out, which is why the choice and the tuner leave such sums to the fp32
// kernels).  With one accumulator, or with truncated parts, it is larger than the chain's for some signs.
//
// What the parts cannot do is done again on the fp32 matrix cores, by the
// waves whose sums it concerns (fp32_sums):
// - An infinite value has a NaN second part, a finite one that rounds to an
//   infinite first part an infinite second part of the other sign, and the
//   leading products of finite values can overflow where their sum does not
//   (their parts round up).  Every such sum comes out as infinity or NaN, and
//   all sums that do are replaced.
// - The parts of some magnitudes below 2^-107 do not add up to the value.  A
//   workgroup that meets one (one instruction a pair of operands tells)
//   replaces all its sums.
//
// The split is done once per loaded element, as it is stored to LDS, in steps
// of a few vector instructions between the matrix-core instructions of the
// slab before it.  What bounds it: the matrix cores are busy 41 to 44% of the
// cycles, 49 to 51% of those in which the compute unit is (256x28x28 -> 256,
// 3x3, 64 images, and AlexNet's conv2; rocprofv3 counters), the rest is barriers
// and LDS latency between slabs, at a clock that bf16 matrix work on random
// data holds at 2.1 GHz (a loop of nothing but these instructions reaches 1.8
// of the nominal 2.5 PFLOP/s).  On 256x28x28 -> 256, 3x3, 64 images: 505 -> 391
// to 402 us (147 to 151 TFLOP/s of the layer's own operations);
// AlexNet at batch 64: 859 -> 738 us on one box, 865 -> 767 on another.
#pragma once

#include <cstring>
#include <type_traits>

#include "bf16_split.h"
#include "conv_igemm_kernel.h"

namespace cnn {
namespace conv {

// Tile element (step, part, row, taps 8 half .. 8 half + 7 of the step): a row
// of a step is 16 bf16 taps (32 bytes), its two 16-byte halves swapped in every
// other group of four rows, so that both the 128-bit fragment reads (eight rows
// of one half at a time) and the 128-bit gather stores touch every bank once.
template <int ROWS>
__device__ inline int tile_at(int step, int part, int row, int half) {
    return ((step * 3 + part) * ROWS + row) * 16 + ((half ^ (row >> 2)) & 1) * 8;
}

// The parts of 8 taps (half of a step) / of 4 taps (quad of a step) of one row;
// each argument holds the three parts of a pair of taps.
template <int ROWS>
__device__ inline void put_oct(unsigned short* tile, int step, int row, int half, const unsigned* a, const unsigned* b,
                               const unsigned* c, const unsigned* d) {
#pragma unroll
    for (int q = 0; q < 3; ++q)
        *reinterpret_cast<uint4*>(tile + tile_at<ROWS>(step, q, row, half)) = make_uint4(a[q], b[q], c[q], d[q]);
}
template <int ROWS>
__device__ inline void put_quad(unsigned short* tile, int step, int row, int quad, const unsigned* a, const unsigned* b) {
#pragma unroll
    for (int q = 0; q < 3; ++q)
        *reinterpret_cast<uint2*>(tile + tile_at<ROWS>(step, q, row, quad >> 1) + (quad & 1) * 4) = make_uint2(a[q], b[q]);
}

// Replaces a wave's FM x FN blocks of sums, all or those that are not finite,
// by sums of the same taps on the fp32 matrix cores (see the header comment).
// kr: this lane's channel (matrix row) of the first block; off, ok: as of
// store_blocks.
template <int FM, int FN>
__device__ inline void fp32_sums(const ConvParams& p, floatx16 (&acc)[FM][FN], bool all, int g, int kr, int half,
                                 const int (&off)[FN], const bool (&ok)[FN], int kbeg, int klen) {
    float nan = 0.0f;  // NaN if a sum is not finite
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) nan = __builtin_fmaf(acc[i][j][v], 0.0f, nan);
    if (!all && !__any(nan != nan)) return;
    const __amdgpu_buffer_rsrc_t xres =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.x), (short)0, p.xbytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t wres =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.w), (short)0, p.wbytes, 0x00020000);
    int h0[FN], w0[FN], img[FN];  // window corner and image group of this lane's pixels
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        const int n = off[j] / (p.K * p.PQ), pq = off[j] - n * p.K * p.PQ;
        const int pp = (int)fdiv(pq, p.f_q);
        h0[j] = pp * p.sh - p.ph;
        w0[j] = (pq - pp * p.Q) * p.sw - p.pw;
        img[j] = (n * p.C + g * p.Cg) * p.HW;
    }
    floatx16 sum[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) sum[i][j][v] = 0.0f;
#pragma unroll 4
    for (int k = half; k < klen + half; k += 2) {  // half: the k index of the instruction
        const int c = (int)fdiv(kbeg + k, p.f_rs);
        const int rs = kbeg + k - c * p.RS;
        const int r = (int)fdiv(rs, p.f_s), s = rs - r * p.S;
        float x[FN], w[FM];
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int h = h0[j] + r, c0 = w0[j] + s;
            const bool in = ok[j] && k < klen && (unsigned)h < (unsigned)p.H && (unsigned)c0 < (unsigned)p.W;
            const int at = in ? (img[j] + c * p.HW + h * p.W + c0) * 4 : kOutOfRange;
            x[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xres, at, 0, 0));
            if (p.relu_x) x[j] = x[j] > 0.0f ? x[j] : 0.0f;
        }
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const bool in = k < klen && kr + i * 32 < p.Kg;
            const int at = in ? ((g * p.Kg + kr + i * 32) * p.Kr + kbeg + k) * 4 : kOutOfRange;
            w[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wres, at, 0, 0));
        }
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
                sum[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[i], x[j], sum[i][j], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const bool keep = !all && __builtin_fabsf(acc[i][j][v]) <= 3.402823466e38f;
                acc[i][j][v] = keep ? acc[i][j][v] : sum[i][j][v];
            }
}

// Bias, ReLU and NCHW store (lanes = consecutive pixels) of a wave's FM x FN
// blocks: channels kr0 + 32 i + ... of group g, and per pixel block j this
// lane's pixel (off[j]: its element offset in channel 0 of y; ok[j]: it
// exists).  The FN pixel blocks of one output channel are stored one after
// the other, so that a channel's run of FN * 32 pixels reaches L2 in
// consecutive instructions (with the blocks stored far apart, 128 x 128 tiles
// on planes that are not a whole number of cache lines wrote 1.36x their
// output to HBM: partial lines written back separately).
template <int FM, int FN>
__device__ inline void store_blocks(const ConvParams& p, const floatx16 (&acc)[FM][FN], int g, int kr0, int half,
                                    const int (&off)[FN], const bool (&ok)[FN]) {
#pragma unroll
    for (int i = 0; i < FM; ++i) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int kr = kr0 + i * 32 + 8 * (v / 4) + 4 * half + (v % 4);
            if (kr >= p.Kg) continue;
            const int ko = g * p.Kg + kr;
            const float bv = (p.splits == 1 && p.bias) ? p.bias[ko] : 0.0f;
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                if (!ok[j]) continue;
                float* dst = p.y + off[j] + ko * p.PQ;
                float val = acc[i][j][v];
                if (p.splits > 1) {
                    atomicAdd(dst, val);
                } else {
                    if (p.bias) val += bv;
                    if (p.relu) val = val > 0.0f ? val : 0.0f;
                    *dst = val;
                }
            }
        }
    }
}

// ST: register stages (slabs of loads in flight).  The compiler is held to two
// or three waves per SIMD: one step of fragments, two sets of accumulators, the
// stages and the parts in flight take 100 to 256 registers a lane, within the
// limit but for configuration 18 with vector weight loads and a tap table (24 to
// 28 bytes of scratch).
template <int WMW, int WNW, int FM, int FN, int BK, bool VEC_W, int GATHER, int ST>
__global__ void __launch_bounds__(64 * WMW * WNW)
__attribute__((amdgpu_waves_per_eu(FM * FN >= 3 || BK == 32 ? 2 : 3)))
conv2d_split_f32(ConvParams p) {
    static_assert(ST % 2 == 0, "the two LDS buffers alternate within a round of ST slabs");
    constexpr int TM = WMW * FM * 32;  // output channels per workgroup
    constexpr int TN = WNW * FN * 32;  // output pixels per workgroup
    constexpr int NT = 64 * WMW * WNW;
    constexpr int KGROUPS = NT / TN;   // threads sharing one pixel column of the gather
    constexpr int KRUN = BK / KGROUPS; // consecutive taps gathered per thread
    constexpr int STEPS = BK / 16;     // matrix-core steps (16 taps) per slab
    static_assert(NT % TN == 0 && TN % 64 == 0, "gather layout needs TN | NT and whole waves per pixel column");
    static_assert(BK % 16 == 0 && KRUN % 4 == 0, "slabs of whole steps, gather runs of whole quads");
    constexpr int WTOT = TM * BK / 4;                  // weight quads (4 taps of a row) per slab
    constexpr int WV = (WTOT + NT - 1) / NT;            // ... per thread
    constexpr int AROWS = WV * NT / (BK / 4);           // TM rows + spare rows

    // LDS: [buffer] weight tiles, then [buffer] im2col tiles, each
    // [step][part][row][16 taps] in bf16 (see tile_at)
    constexpr int A_ELEMS = STEPS * 3 * AROWS * 16, B_ELEMS = STEPS * 3 * TN * 16;
    __shared__ __attribute__((aligned(16))) unsigned short smem[2 * (A_ELEMS + B_ELEMS)];
    __shared__ int any_lost;  // an operand of the workgroup did not split
    if (threadIdx.x == 0) any_lost = 0;

    const int tid = threadIdx.x;
    auto sA = [&](int buf) { return smem + buf * A_ELEMS; };
    auto sB = [&](int buf) { return smem + 2 * A_ELEMS + buf * B_ELEMS; };
    const int g = blockIdx.z % p.G;
    const int kbeg = (blockIdx.z / p.G) * p.kchunk;  // first tap of this chunk
    const int klen = min(p.kchunk, p.Kr - kbeg);      // taps in this chunk
    // Workgroup -> tile.  A launch's workgroups go to the 8 XCDs in turn by
    // linear id, and each XCD has its own L2: the tiles that read the same
    // input (every channel tile of a pixel tile, and neighbouring pixel
    // tiles, whose windows overlap) are given to workgroups of one XCD, in
    // channel-tile-fastest order.  Ids past the last multiple of 8 keep their
    // position.
    int m0, k0;
    {
        const int gy = gridDim.y;
        const int tiles = gridDim.x * gy;
        const int wg = blockIdx.x + gridDim.x * blockIdx.y;
        const int full = tiles & ~7;
        const int seq = wg < full ? (wg & 7) * (full >> 3) + (wg >> 3) : wg;
        m0 = (seq / gy) * TN;
        k0 = (seq % gy) * TM;
    }

    // ---- gather setup: this thread's pixel and tap run (fixed for all slabs)
    const int mloc = tid % TN;
    const int kgrp = __builtin_amdgcn_readfirstlane(tid / TN);  // uniform: TN is a multiple of 64
    const int m = m0 + mloc;
    int hb, wb, lane_off;
    if (m < p.M) {
        const int n = (int)fdiv(m, p.f_pq);
        const int pq = m - n * p.PQ;
        const int pp = (int)fdiv(pq, p.f_q);
        const int qq = pq - pp * p.Q;
        hb = pp * p.sh - p.ph;
        wb = qq * p.sw - p.pw;
        lane_off = ((n * p.C + g * p.Cg) * p.HW + hb * p.W + wb) * 4;
    } else {
        hb = -0x40000000;  // every row test fails: the column reads as zero
        wb = 0;
        lane_off = 0;
    }
    const __amdgpu_buffer_rsrc_t xres =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.x), (short)0, p.xbytes, 0x00020000);

    const int niter = (klen + BK - 1) / BK;  // slabs
    extern __shared__ __attribute__((aligned(16))) int stab[];  // (niter + ST) * BK entries
    unsigned inv = 0xffffffffu;
    if constexpr (GATHER != kGatherScalar) {
        for (int kk = threadIdx.x; kk < (niter + ST) * BK; kk += NT) {
            int e = GATHER == kGatherMask ? 31 : GATHER == kGatherStridedMask ? 63 : (int)0x80000000u;
            if (kk < klen) {
                const int c = (int)fdiv(kbeg + kk, p.f_rs);
                const int rs = kbeg + kk - c * p.RS;
                const int r = (int)fdiv(rs, p.f_s);
                const int s = rs - r * p.S;
                const int toff = ((c * p.H + r) * p.W + s) * 4;
                e = GATHER == kGatherMask ? ((toff << 5) | rs) : GATHER == kGatherStridedMask ? ((toff << 6) | rs) : toff;
            }
            stab[kk] = e;
        }
        if (GATHER == kGatherNoPad && m >= p.M) lane_off = (int)0x80000000u;
    }
    if constexpr (GATHER == kGatherMask) {
        if (m < p.M) inv = 0x80000000u | outside_taps<unsigned>(hb, wb, p.H, p.W, p.R, p.S);
    }
    // strided gather: element u of a thread is pixel group u / TG (16 pixels
    // apart) and tap group u % TG (4 taps apart) of its wave's pixels
    constexpr int TG = BK / 4;          // tap groups per slab
    constexpr int PPT = KRUN / TG;      // pixels per thread
    constexpr int PW = 16 * PPT;        // pixels per wave
    constexpr bool STRIDED = GATHER == kGatherStrided || GATHER == kGatherStridedMask;
    static_assert(!STRIDED || (KRUN % TG == 0 && (NT / 64) * PW == TN),
                  "strided gather: whole pixel groups per wave");
    const int ln = tid & 63;
    const int wpix = (tid >> 6) * PW + (ln >> 2);  // this thread's first pixel, within the tile
    int soff[STRIDED ? PPT : 1];
    unsigned long long inv64[GATHER == kGatherStridedMask ? PPT : 1];
    if constexpr (STRIDED) {
#pragma unroll
        for (int pi = 0; pi < PPT; ++pi) {
            const int mm = m0 + wpix + pi * 16;
            inv64[GATHER == kGatherStridedMask ? pi : 0] = ~0ull;
            if (mm < p.M) {
                const int n = (int)fdiv(mm, p.f_pq);
                const int pq = mm - n * p.PQ;
                const int pp = (int)fdiv(pq, p.f_q);
                const int qq = pq - pp * p.Q;
                const int h0 = pp * p.sh - p.ph, w0 = qq * p.sw - p.pw;
                soff[pi] = ((n * p.C + g * p.Cg) * p.HW + h0 * p.W + w0) * 4;
                if constexpr (GATHER == kGatherStridedMask)
                    inv64[pi] = (1ull << 63) | outside_taps<unsigned long long>(h0, w0, p.H, p.W, p.R, p.S);
            } else {
                soff[pi] = GATHER == kGatherStridedMask ? 0 : (int)0x80000000u;
            }
        }
    }
    if constexpr (GATHER != kGatherScalar) __syncthreads();

    // Table entries of a slab's elements, then one load per element u of this
    // thread (STRIDED: pixel group u / TG, tap group u % TG).
    constexpr int NTAB = GATHER == kGatherScalar ? 1 : STRIDED ? TG : KRUN;
    int tab[NTAB];
    auto read_tab = [&](int kslab) {
        if constexpr (STRIDED) {
#pragma unroll
            for (int q = 0; q < TG; ++q) tab[q] = stab[kslab + 4 * q + (ln & 3)];
        } else if constexpr (GATHER != kGatherScalar) {
#pragma unroll
            for (int j = 0; j < KRUN; j += 4) {
                const int4 e4 = *reinterpret_cast<const int4*>(&stab[kslab + kgrp * KRUN + j]);
                tab[j] = e4.x, tab[j + 1] = e4.y, tab[j + 2] = e4.z, tab[j + 3] = e4.w;
            }
        }
    };
    float xr[ST][KRUN];  // register stages
    auto load_x1 = [&](int sg, int u) {
        int voff;
        if constexpr (STRIDED) {
            const int e = tab[u % TG];
            if constexpr (GATHER == kGatherStridedMask) {
                const unsigned bad = (unsigned)(inv64[u / TG] >> (e & 63)) & 1u;
                voff = (soff[u / TG] + (e >> 6)) | (int)(bad << 31);
            } else {
                voff = (int)((unsigned)soff[u / TG] + (unsigned)e);
            }
        } else if constexpr (GATHER == kGatherMask) {
            const unsigned e = (unsigned)tab[u];
            voff = (lane_off + (int)(e >> 5)) | (int)(((inv >> (e & 31)) & 1u) << 31);
        } else {
            voff = (int)((unsigned)lane_off + (unsigned)tab[u]);
        }
        xr[sg][u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xres, voff, 0, 0));
    };
    auto load_x_scalar = [&](int kslab, int sg) {
        const int kk0 = kslab + kgrp * KRUN;  // uniform
        const int ka0 = kbeg + kk0;           // absolute tap index
        int c = (int)fdiv(ka0, p.f_rs);
        const int rs = ka0 - c * p.RS;
        int r = (int)fdiv(rs, p.f_s);
        int s = rs - r * p.S;
        int toff = ((c * p.H + r) * p.W + s) * 4;  // byte offset of tap (c, r, s)
#pragma unroll
        for (int j = 0; j < KRUN; ++j) {
            const bool ok = (kk0 + j < klen) && ((unsigned)(hb + r) < (unsigned)p.H) &&
                            ((unsigned)(wb + s) < (unsigned)p.W);
            const int voff = ok ? lane_off + toff : kOutOfRange;
            xr[sg][j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xres, voff, 0, 0));
            // next tap: s, then r, then c
            ++s;
            toff += 4;
            const bool wrap_s = (s == p.S);
            s = wrap_s ? 0 : s;
            r += wrap_s ? 1 : 0;
            toff += wrap_s ? (p.W - p.S) * 4 : 0;
            const bool wrap_r = (r == p.R);
            r = wrap_r ? 0 : r;
            toff += wrap_r ? (p.HW - p.R * p.W) * 4 : 0;
        }
    };

    // ---- weight tile loads: rows k0.. of the group's [Kg][Kr] block, through a
    // buffer resource as well (rows past the group or taps past the reduction
    // read as zero).  Items past the tile land in spare LDS rows never read.
    const __amdgpu_buffer_rsrc_t wres =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.w), (short)0, p.wbytes, 0x00020000);
    int w_off[WV], w_col[WV], w_row[WV];
    bool w_rowok[WV];
    constexpr bool WQUAD = VEC_W && !STRIDED;  // one 128-bit load per quad
    constexpr int WSTEP = STRIDED ? 4 : 1;     // distance of a quad's taps in the reduction
#pragma unroll
    for (int i = 0; i < WV; ++i) {
        const int idx = tid + i * NT;
        w_row[i] = idx / (BK / 4);
        w_col[i] = idx % (BK / 4);  // quad within the slab
        w_rowok[i] = w_row[i] < TM && k0 + w_row[i] < p.Kg;
        // first tap of the quad within the slab
        const int tap = STRIDED ? (w_col[i] & ~3) * 4 + (w_col[i] & 3) : w_col[i] * 4;
        w_off[i] = w_rowok[i] ? ((g * p.Kg + k0 + w_row[i]) * p.Kr + kbeg + tap) * 4 : 0;
    }
    float wr[ST][WV * 4];
    constexpr int WLOADS = WV * (WQUAD ? 1 : 4);
    auto load_w1 = [&](int kslab, int sg, int l) {
        const int i = WQUAD ? l : l / 4, u = WQUAD ? 0 : l % 4;
        const int tap = STRIDED ? (w_col[i] & ~3) * 4 + (w_col[i] & 3) : w_col[i] * 4;
        const bool ok = w_rowok[i] && (kslab + tap + u * WSTEP < klen);
        const int voff = ok ? w_off[i] + (kslab + u * WSTEP) * 4 : kOutOfRange;
        if constexpr (WQUAD) {
            // Cast the whole vector: a bit-cast of one element of an
            // ext_vector lvalue reads element 0 with this compiler.
            typedef float f32x4 __attribute__((ext_vector_type(4)));
            const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(wres, voff, 0, 0));
#pragma unroll
            for (int e = 0; e < 4; ++e) wr[sg][4 * i + e] = v[e];
        } else {
            wr[sg][4 * i + u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wres, voff, 0, 0));
        }
    };

    // ---- split and store of a slab's loads, in SIDE steps of a few vector
    // instructions each, to be placed between matrix-core instructions: step
    // 3 i + q makes part q of element pair i (the gather's pairs, then the
    // weights') and stores the parts of a quad or oct once its last pair is done.
    constexpr int XPAIRS = KRUN / 2, PAIRS = XPAIRS + 2 * WV, SIDE = 3 * PAIRS;
    unsigned part[PAIRS][3];
    unsigned lost = 0;  // whether an operand did not split (note_lost)
    auto side_step = [&](auto relu, int buf, int sg, int step) {
        const int i = step / 3, q = step % 3;
        float* v = i < XPAIRS ? &xr[sg][2 * i] : &wr[sg][2 * (i - XPAIRS)];
        if constexpr (decltype(relu)::value)
            if (i < XPAIRS && q == 0) {
                v[0] = v[0] > 0.0f ? v[0] : 0.0f;
                v[1] = v[1] > 0.0f ? v[1] : 0.0f;
            }
        if (q == 2) note_lost(lost, v);
        part[i][q] = split_step(v, q < 2);
        if (q < 2) return;
        if (i >= XPAIRS) {
            if (i % 2 != (XPAIRS + 1) % 2) return;
            const int l = (i - XPAIRS) / 2;
            put_quad<AROWS>(sA(buf), w_col[l] >> 2, w_row[l], w_col[l] & 3, part[i - 1], part[i]);
        } else if (STRIDED) {
            // tap 4q + t of a step is kept at position 4t + q (the weights
            // likewise), so that the four taps this thread holds of a step are
            // neighbours
            if (i % 2 != 1) return;
            const int u = 2 * i - 2;  // element of the quad's first tap
            put_quad<TN>(sB(buf), u % TG / 4, wpix + u / TG * 16, ln & 3, part[i - 1], part[i]);
        } else if (KRUN % 8 == 0) {
            if (i % 4 != 3) return;
            const int pos = kgrp * KRUN + 2 * i - 6;
            put_oct<TN>(sB(buf), pos >> 4, mloc, (pos >> 3) & 1, part[i - 3], part[i - 2], part[i - 1], part[i]);
        } else {
            if (i % 2 != 1) return;
            const int pos = kgrp * KRUN + 2 * i - 2;
            put_quad<TN>(sB(buf), pos >> 4, mloc, (pos >> 2) & 3, part[i - 1], part[i]);
        }
    };

    // ---- matrix-core work of one slab
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave / WNW;
    const int wn = wave % WNW;
    const int half = lane >> 5;
    const int l32 = lane & 31;
    floatx16 acc[FM][FN], low[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = low[i][j][v] = 0.0f;

    // side(q) is called after matrix-core instruction q of the slab
    constexpr int NM = 6 * FM * FN * STEPS;
    auto compute = [&](int buf, auto side) {
        bf16x8 a[STEPS][3][FM], b[STEPS][3][FN];
#pragma unroll
        for (int st = 0; st < STEPS; ++st)
#pragma unroll
            for (int q = 0; q < 3; ++q) {
#pragma unroll
                for (int i = 0; i < FM; ++i)
                    a[st][q][i] = *reinterpret_cast<const bf16x8*>(
                        sA(buf) + tile_at<AROWS>(st, q, wm * FM * 32 + i * 32 + l32, half));
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    b[st][q][j] = *reinterpret_cast<const bf16x8*>(
                        sB(buf) + tile_at<TN>(st, q, wn * FN * 32 + j * 32 + l32, half));
            }
        // the six products of parts above 2^-24 of the whole
        constexpr int PA[6] = {0, 0, 1, 1, 0, 2}, PB[6] = {0, 1, 0, 1, 2, 0};
#pragma unroll
        for (int st = 0; st < STEPS; ++st)
#pragma unroll
            for (int q = 0; q < 6; ++q)
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j) {
                        floatx16& c = q == 0 ? acc[i][j] : low[i][j];
                        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[st][PA[q]][i], b[st][PB[q]][j], c, 0, 0, 0);
                        side(((st * 6 + q) * FM + i) * FN + j);
                    }
    };

    // ---- main loop.  ST slabs of loads are in flight (ST register stages).
    // While slab s is multiplied from LDS buffer s % 2, slab s + 1 is split from
    // stage (s + 1) % ST into the other buffer and slab s + ST requested into
    // the freed stage s % ST.  One barrier per slab: it publishes slab s, and
    // nobody reads buffer (s + 1) % 2 (slab s - 1) after it.  The last
    // niter % ST slabs run after the loop, so that the loop body is
    // straight-line code and each split waits only for its own loads.
    auto load = [&](int kslab, int sg) {
        if constexpr (GATHER == kGatherScalar) {
            load_x_scalar(kslab, sg);
        } else {
            read_tab(kslab);
#pragma unroll
            for (int u = 0; u < KRUN; ++u) load_x1(sg, u);
        }
#pragma unroll
        for (int l = 0; l < WLOADS; ++l) load_w1(kslab, sg, l);
    };
    auto store = [&](auto relu, int buf, int sg) {
#pragma unroll
        for (int t = 0; t < SIDE; ++t) side_step(relu, buf, sg, t);
    };
    auto reduce = [&](auto relu) {
#pragma unroll
        for (int j = 0; j < ST; ++j) load(j * BK, j);
        store(relu, 0, 0);
        int it = 0;
        for (; it + ST - 1 < niter; it += ST) {
#pragma unroll
            for (int j = 0; j < ST; ++j) {
                const int next = (it + j + ST) * BK;
                __syncthreads();
                if constexpr (GATHER == kGatherScalar) load_x_scalar(next, j);
                else read_tab(next);
                constexpr int XLOADS = GATHER == kGatherScalar ? 0 : KRUN, LOADS = XLOADS + WLOADS;
                compute(j & 1, [&](int q) {
#pragma unroll
                    for (int t = q * SIDE / NM; t < (q + 1) * SIDE / NM; ++t)
                        side_step(relu, (j + 1) & 1, (j + 1) % ST, t);
#pragma unroll
                    for (int l = q * LOADS / NM; l < (q + 1) * LOADS / NM; ++l) {
                        if (l < XLOADS) load_x1(j, l);
                        else load_w1(next, j, l - XLOADS);
                    }
                    // The strided gathers keep the compiler's order, as in
                    // conv_igemm_kernel.h: there a pinned order returned a tap
                    // as zero when workgroups shared a compute unit, for a
                    // reason that was not established.
                    if constexpr (!STRIDED) __builtin_amdgcn_sched_barrier(0);
                });
            }
        }
#pragma unroll
        for (int j = 0; j < ST - 1; ++j) {
            if (it + j < niter) {
                __syncthreads();
                if (it + j + 1 < niter) store(relu, (j + 1) & 1, (j + 1) % ST);
                compute(j & 1, [](int) {});
            }
        }
    };
    if (p.relu_x) reduce(std::true_type{});
    else reduce(std::false_type{});
    if (split_lost(lost)) any_lost = 1;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] += low[i][j][v];
    // ---- epilogue
    int off[FN];
    bool ok[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        const int mc = m0 + wn * FN * 32 + j * 32 + l32;
        ok[j] = mc < p.M;
        const int n = ok[j] ? (int)fdiv(mc, p.f_pq) : 0;
        off[j] = ok[j] ? n * p.K * p.PQ + mc - n * p.PQ : 0;
    }
    const int kr0 = k0 + wm * FM * 32;
    __syncthreads();
    fp32_sums<FM, FN>(p, acc, any_lost != 0, g, kr0 + l32, half, off, ok, kbeg, klen);
    store_blocks<FM, FN>(p, acc, g, kr0, half, off, ok);
}

template <int WMW, int WNW, int FM, int FN, int BK, int ST, bool VEC_W, int GATHER>
inline void launch_split_kernel(const ConvParams& prm, dim3 grid, dim3 block, size_t shm, hipStream_t st) {
    enqueue((conv2d_split_f32<WMW, WNW, FM, FN, BK, VEC_W, GATHER, ST>), grid, block, shm, st, prm);
}

// Picks the gather mode for the shape and launches one configuration.
template <int WMW, int WNW, int FM, int FN, int BK, int ST>
int launch_split(const ConvParams& prm, bool vec_w, hipStream_t st) {
    constexpr int TM = WMW * FM * 32;
    constexpr int TN = WNW * FN * 32;
    dim3 grid(ceil_div(prm.M, TN), ceil_div(prm.Kg, TM), prm.G * prm.splits);
    dim3 block(64 * WMW * WNW);
    // tap tables are at most 32 KiB of LDS
    const int tab_entries = (ceil_div(prm.kchunk, BK) + ST) * BK;
    const bool tab_fits = tab_entries * 4 <= 32768;
    int mode = kGatherScalar;
    if (tab_fits && prm.ph == 0 && prm.pw == 0)
        mode = prm.sw > 1 ? kGatherStrided : kGatherNoPad;
    else if (tab_fits && prm.sw > 1 && prm.RS <= 63 && (int64_t)prm.Cg * prm.HW * 4 < ((int64_t)1 << 25))
        mode = kGatherStridedMask;
    else if (tab_fits && prm.RS <= 31 && (int64_t)prm.Cg * prm.HW * 4 < ((int64_t)1 << 27))
        mode = kGatherMask;
    const size_t shm = mode == kGatherScalar ? 0 : (size_t)tab_entries * 4;
    // the strided gathers load weights tap by tap whatever the rows' alignment
#define GO(V, M) launch_split_kernel<WMW, WNW, FM, FN, BK, ST, V, M>(prm, grid, block, shm, st)
    if (mode == kGatherStridedMask) GO(false, kGatherStridedMask);
    else if (mode == kGatherStrided) GO(false, kGatherStrided);
    else if (vec_w) {
        if (mode == kGatherNoPad) GO(true, kGatherNoPad);
        else if (mode == kGatherMask) GO(true, kGatherMask);
        else GO(true, kGatherScalar);
    } else {
        if (mode == kGatherNoPad) GO(false, kGatherNoPad);
        else if (mode == kGatherMask) GO(false, kGatherMask);
        else GO(false, kGatherScalar);
    }
#undef GO
    return check_launch("conv2d_split_f32");
}

// Defines launch_c<I> of a split configuration.
#define CNN_SPLIT_DEFINE(I, WMW, WNW, FM, FN, BK)                                  \
    int launch_c##I(const ConvParams& prm, bool vec_w, hipStream_t st) {           \
        return launch_split<WMW, WNW, FM, FN, BK, 2>(prm, vec_w, st);           \
    }

}  // namespace conv
}  // namespace cnn
