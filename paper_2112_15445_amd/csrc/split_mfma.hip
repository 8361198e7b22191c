// SC_F32 on the matrix cores (SLAB tunings with pipeline = 3): the densified layer with every fp32
// operand split into three bfloat16 terms.
//
// An fp32 value is exactly x = hi + mid + lo with hi the bfloat16 nearest to x, mid the one nearest to
// x - hi and lo the rest, which fits a bfloat16: 8 significant bits each (the splitting of Henry, Tang and
// Heinecke, "Leveraging the bfloat16 artificial intelligence datatype for higher-precision computations",
// 2019).  With x in [2^e, 2^(e+1)), |mid| is at most 2^(e-8) and |lo| at most 2^(e-17).  A product is then the sum
// of nine exact products, of which the six largest are kept: mid lo and lo mid are at most 2^-25 of it each, lo lo
// 2^-34.  That is as much as one rounding of a fused multiply-add, of which the gather kernels do one per stored
// weight and this form one per 32 channels of a tap, so it counts where the rows are short: tables with a row of
// 1 .. 15 weights keep mid lo and lo mid too (FULL; as a template parameter: a branch on it in the
// multiplication costs the others 10 %).  (With hi truncated instead, mid lo and lo mid reach 2^-22 of
// the product together, and all eight have to be kept: 45.7 us for 39.8 on the 3x3 128-128 layer at 28 x 28, batch 32.)
// Each product is one v_mfma_f32_16x16x32_bf16 over 32 input channels of one filter tap,
// accumulated in fp32: hi hi in one set of accumulators, the small ones in a second set (their
// roundings are 2^-7 of the first set's), added once at the end.  The sum over a row is rounded
// once per 32 channels of a tap instead of once per stored entry, which is why the result is
// closer to the exact one than the gather kernels' (relative error against 64 bits 5e-8 .. 1e-7 where theirs is 0.9e-7 .. 3.7e-7).
// Bound by the matrix pipes: 6 instructions per 16 x 16 x 32 block, at the 1.8 - 1.9 PFLOP/s that
// the 16 x 16 x 32 bfloat16 instruction sustains with two waves per SIMD (1.24 with one, which is
// why the workgroups that do not share a CU have eight waves) about 300 TFLOP/s of fp32 products,
// against 154 of the fp32 matrix instructions and 78 of the vector units without packed math.
//
// The terms hold a value's 24 bits only down to 2^-110 (the last bit of lo is then the smallest bfloat16), and a
// product's small terms need room above the smallest fp32: an output may be off by n (2^-133 of the largest weight +
// 2^-147).  At the other end a hi is infinite from 2^128 - 2^119 on, and an infinite input meets zeros that the
// sparse table does not hold: either leaves NaN in every output that the tile computes from that place.  A
// wave that has an output below 2^28 of that error (a.floor) but not zero, or one that is not finite, therefore sums
// its outputs entry by entry from the sparse table instead (split_exact): the gather kernels' result.  Ordinary
// activations never get there; the test of the outputs is one and a half vector instructions each.  (Noting small inputs
// while they are staged, the first form of this, was three for every pair of inputs and cost 0.7 us on the 1-D
// 300-64 layer.)  What is left: an output all of whose inputs but zeros are 2^-134 or less comes out as zero.
//
// Tile, staging, weight order and step order are those of the DENSE variant (dense_mfma.hip): a
// workgroup owns DB output channels x a tile of positions; the input region of the tile is staged
// channel-minor in LDS, here as three bfloat16 images, split on the way; weights are split and put
// in operand order once per plan.
#include <algorithm>
#include <cstring>

#include "dense_mfma_kernel.h"

namespace sc {

struct SplitArgs {
    unsigned floor;          // 2 bits(m) + 2^24 of the smallest magnitude m of an output that the terms serve
    int C, D, N, H, W, P, Q, S, RS, s_h, s_w, pad_h, pad_w;
    int TP, NS, tiles_p, Hs, Ws, npos_s, npos, CC, nchunks, NCB, pitch, bufsz, DB, ndb, epv, TPQ;
    int cbs_last;            // channel blocks of the last chunk
    int KS, cps;             // workgroups that share the chunks of a tile, chunks for each
    int npos1;               // staged positions of one sample (Hs * Ws)
    int flat;                // the staged rows of a sample are one contiguous run per channel
    int wmajor, ntiles;      // output-channel blocks outermost; (sample group, row tile) pairs
    float inv_ntiles, inv_KS, inv_ndb, inv_tiles_p, inv_HsWs, inv_Ws, inv_TPQ, inv_Q;
    int n;                   // the sparse table, for split_exact
    const float* theta;
    const int32_t *col, *len;
};

typedef __bf16 bf8v __attribute__((ext_vector_type(8)));

typedef __bf16 bf2v __attribute__((ext_vector_type(2)));
typedef float float2v __attribute__((ext_vector_type(2)));

// The three terms of two values, packed as bfloat16 pairs (the first value in the low half): 11
// vector instructions.
__device__ __forceinline__ void split3x2(float x0, float x1, unsigned& hi, unsigned& mid, unsigned& lo)
{
    hi = __builtin_bit_cast(unsigned, __builtin_convertvector((float2v){x0, x1}, bf2v));                    // to nearest
    const float r0 = x0 - __uint_as_float(hi << 16), r1 = x1 - __uint_as_float(hi & 0xffff0000u);           // exact
    mid = __builtin_bit_cast(unsigned, __builtin_convertvector((float2v){r0, r1}, bf2v));                   // to nearest
    const float l0 = r0 - __uint_as_float(mid << 16), l1 = r1 - __uint_as_float(mid & 0xffff0000u);         // exact
    lo = __builtin_amdgcn_perm(__float_as_uint(l1), __float_as_uint(l0), 0x07060302u);                      // exact: the upper halves
}

// One block of positions times MW blocks of output channels: six matrix instructions for each, eight with
// FULL, the smallest products first.
template <bool FULL, int MW, int NW>
__device__ __forceinline__ void split_multiply(float4v (&acc)[MW][NW], float4v (&accs)[MW][NW], const uint4w (&av)[MW][3],
                                               const uint4w (&bv)[3], int i)
{
    auto mul = [&](float4v& c, const uint4w& a, const uint4w& b) {
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8v, a), __builtin_bit_cast(bf8v, b), c, 0, 0, 0);
    };
    if constexpr (FULL) {
#pragma unroll
        for (int m = 0; m < MW; ++m) mul(accs[m][i], av[m][1], bv[2]);
#pragma unroll
        for (int m = 0; m < MW; ++m) mul(accs[m][i], av[m][2], bv[1]);
    }
#pragma unroll
    for (int m = 0; m < MW; ++m) mul(accs[m][i], av[m][0], bv[2]);
#pragma unroll
    for (int m = 0; m < MW; ++m) mul(acc[m][i], av[m][0], bv[0]);
#pragma unroll
    for (int m = 0; m < MW; ++m) mul(accs[m][i], av[m][2], bv[0]);
#pragma unroll
    for (int m = 0; m < MW; ++m) mul(accs[m][i], av[m][1], bv[1]);
#pragma unroll
    for (int m = 0; m < MW; ++m) mul(accs[m][i], av[m][0], bv[1]);
#pragma unroll
    for (int m = 0; m < MW; ++m) mul(accs[m][i], av[m][1], bv[0]);
}

// floor(e / d) as fdiv19, one fused multiply-add (e < 2^19; inv within an ulp of 1 / d)
__device__ __forceinline__ int sdiv(int e, float inv) { return (int)__builtin_fmaf((float)e, inv, 0.5f * inv); }
// (full 32-bit multiplies run at a quarter of the rate: products that fit 24-bit factors use these)
__device__ __forceinline__ int mul24(int p, int q) { return __mul24(p, q); }

// ------------------------------------------------------------------------------------------------
// Weights: the layout of the DENSE variant's array with three operand blocks (hi, mid, lo) of 1 KB
// per (16 output channels, tap, 32 input channels).
// ------------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
densify_split_kernel(const float* __restrict__ theta, const int32_t* __restrict__ col, const int32_t* __restrict__ len,
                     unsigned char* __restrict__ out, int D, int n, int RS, int NCB)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)D * n) return;
    const int d = (int)(i / n), j = (int)(i - (int64_t)d * n);
    if (j >= len[d]) return;
    const int k = col[i] & 0x7fffffff;
    const int c = k / RS, tap = k - c * RS;
    const int cblk = c >> 5, cin = c & 31;
    const int64_t blk = (((int64_t)(d >> 4) * RS + tap) * NCB + cblk) * 3;
    unsigned short* dst = reinterpret_cast<unsigned short*>(out + blk * 1024 + ((d & 15) + 16 * (cin >> 3)) * 16) + (cin & 7);
    unsigned h, m, l;
    split3x2(theta[i], 0.0f, h, m, l);
    dst[0] = (unsigned short)h;
    dst[512] = (unsigned short)m;
    dst[1024] = (unsigned short)l;
}

size_t split_weight_bytes(const Plan& p)
{
    const int64_t NCB = (p.L.C + 31) / 32;
    const int64_t rows16 = (int64_t)((p.L.D + 127) / 128) * 8;          // (whole blocks of 128: every operand load is in bounds)
    return (size_t)(rows16 * p.L.R * p.L.S * NCB * 3 * 1024);
}

sc_status_t split_densify(const Plan& p, unsigned char* out, hipStream_t stream)
{
    const int64_t cnt = (int64_t)p.L.D * p.n;
    if (hipMemsetAsync(out, 0, split_weight_bytes(p), stream) != hipSuccess) return SC_ERR_HIP;
    if (cnt == 0) return SC_OK;
    hipLaunchKernelGGL(densify_split_kernel, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, stream,
                       static_cast<const float*>(p.d_theta), p.d_col, p.d_len, out, p.L.D, p.n, p.L.R * p.L.S, (p.L.C + 31) / 32);
    return hipGetLastError() == hipSuccess ? SC_OK : SC_ERR_HIP;
}

// ------------------------------------------------------------------------------------------------
// Staging of one chunk: blocks of 8 channels x EPV columns, the widest loads the runs allow, split
// and transposed in registers, one 16-byte word per position, channel group and image.  `rows` runs
// of `run` elements per sample and channel (where the staged rows carry no padding columns they are
// one run).  Blocks are dealt to the threads in rounds; a round is 32 registers of loads per thread.
// The first round of the next chunk is loaded before the current one is multiplied (load_round,
// then store_round behind the multiplication), so that small chunks cost no memory latency.
// ------------------------------------------------------------------------------------------------
struct SplitRows {
    int nsv;               // samples of this workgroup inside the batch
    int ilo, nrows;        // staged rows that lie inside the input: [ilo, ilo + nrows)
    int rlo;               // input row of staged row ilo
    int wcols;             // input columns that are staged: [0, wcols)
};

// padding: staged positions outside the input or past the batch are zeros in all three images
__device__ __forceinline__ void split_pad(unsigned char* lds, int tid, int NT, int cgroups, const SplitRows& sa, const SplitArgs& a)
{
    // (a layer without padding needs none: a position past the batch or the plane feeds only itself)
    if (!a.pad_h && !a.pad_w) return;
    for (int pos = tid; pos < a.npos_s; pos += NT) {
        const int sm = sdiv(pos, a.inv_HsWs);
        const int rem = pos - mul24(sm, a.npos1);
        const int i = sdiv(rem, a.inv_Ws);
        const int w = rem - mul24(i, a.Ws);
        const bool inside = sm < sa.nsv && i >= sa.ilo && i < sa.ilo + sa.nrows && w >= a.pad_w && w < a.pad_w + sa.wcols;
        if (!inside)
            for (int t = 0; t < 3; ++t)
                for (int cg = 0; cg < cgroups; ++cg) *reinterpret_cast<uint4w*>(lds + t * a.bufsz + mul24(pos, a.pitch) + cg * 16) = uint4w{0u, 0u, 0u, 0u};
    }
}

struct SplitStage {
    const char* xs;        // first staged element of sample 0, channel 0 of the chunk
    unsigned sample4, plane4, row4;    // bytes per sample, channel and input row
    int nblocks, rowsG, per_cg, G, run, cleft, dst0;
    bool whole;            // every channel of the chunk's groups exists in the layer
    float inv_per_cg, inv_rowsG, inv_G;
};

template <int EPV>
__device__ __forceinline__ bool split_block(const SplitStage& st, int v, int& cg, int& sm, int& ii, int& g)
{
    const bool live = v < st.nblocks;
    const int vv = live ? v : 0;                           // (past the end: block 0 again, not written)
    cg = sdiv(vv, st.inv_per_cg);
    const int rb = vv - mul24(cg, st.per_cg);
    sm = 0;
    int r2 = rb;
    if (st.rowsG != st.per_cg) { sm = sdiv(rb, st.inv_rowsG); r2 = rb - mul24(sm, st.rowsG); }
    ii = 0;
    g = r2;
    if (st.rowsG != st.G) { ii = sdiv(r2, st.inv_G); g = r2 - mul24(ii, st.G); }
    return live;
}

template <int EPV>
__device__ __forceinline__ void load_round(float (&pre)[32], const SplitStage& st, int v0, int NT)
{
    constexpr int VB = 4 / EPV;
    struct alignas(EPV * 4) Vec { float e[EPV]; };
#pragma unroll
    for (int u = 0; u < VB; ++u) {
        int cg, sm, ii, g;
        split_block<EPV>(st, v0 + u * NT, cg, sm, ii, g);
        // (32-bit offsets from a wave-uniform base: one address register per load)
        unsigned off = (unsigned)mul24(ii, (int)st.row4) + g * (EPV * 4);
        if (st.rowsG != st.per_cg) off += sm * st.sample4;
        unsigned o = off + cg * (8 * st.plane4);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            // (channels past the layer's last: the block's place in channel 0, zeroed when it is stored)
            const Vec t = *reinterpret_cast<const Vec*>(st.xs + (st.whole || cg * 8 + j < st.cleft ? o : off));
#pragma unroll
            for (int e = 0; e < EPV; ++e) pre[(u * 8 + j) * EPV + e] = t.e[e];
            o += st.plane4;
        }
    }
}

template <int EPV>
__device__ __forceinline__ void store_round(const float (&pre)[32], const SplitStage& st, unsigned char* lds, int v0, int NT, const SplitArgs& a)
{
    constexpr int VB = 4 / EPV;
#pragma unroll
    for (int u = 0; u < VB; ++u) {
        int cg, sm, ii, g;
        if (!split_block<EPV>(st, v0 + u * NT, cg, sm, ii, g)) continue;
        unsigned char* dst = lds + mul24(mul24(sm, a.npos1) + st.dst0 + mul24(ii, a.Ws) + g * EPV, a.pitch) + cg * 16;
        const int left = st.run - g * EPV;                 // columns of this block that are staged
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
            if (e >= left) continue;
            uint4w w0, w1, w2;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v0 = pre[(u * 8 + 2 * q) * EPV + e], v1 = pre[(u * 8 + 2 * q + 1) * EPV + e];
                if (!st.whole) {
                    if (cg * 8 + 2 * q >= st.cleft) v0 = 0.0f;
                    if (cg * 8 + 2 * q + 1 >= st.cleft) v1 = 0.0f;
                }
                unsigned t0, t1, t2;
                split3x2(v0, v1, t0, t1, t2);
                w0[q] = t0; w1[q] = t1; w2[q] = t2;
            }
            *reinterpret_cast<uint4w*>(dst + e * a.pitch) = w0;
            *reinterpret_cast<uint4w*>(dst + e * a.pitch + a.bufsz) = w1;
            *reinterpret_cast<uint4w*>(dst + e * a.pitch + 2 * a.bufsz) = w2;
            __builtin_amdgcn_sched_barrier(0);                 // (one column's terms at a time: registers)
        }
    }
}

// One output entry by entry, in the order of the gather kernels, over the input channels [c_lo, c_hi).
__device__ __forceinline__ float split_exact(const float* __restrict__ x, const SplitArgs& a, int b, int d, int p, int q, int c_lo, int c_hi)
{
    const int i0 = p * a.s_h - a.pad_h, w0 = q * a.s_w - a.pad_w;
    const float* xb = x + (int64_t)b * a.C * a.H * a.W;
    float sum = 0.0f;
#pragma unroll 1
    for (int j = 0; j < a.len[d]; ++j) {
        const int64_t at = (int64_t)d * a.n + j;
        const int k = a.col[at] & 0x7fffffff, c = k / a.RS, tap = k - c * a.RS, r = tap / a.S;
        const int i = i0 + r, w = w0 + tap - r * a.S;
        if (c >= c_lo && c < c_hi && i >= 0 && i < a.H && w >= 0 && w < a.W)
            sum = __builtin_fmaf(a.theta[at], xb[((int64_t)c * a.H + i) * a.W + w], sum);
    }
    return sum;
}

// The wave's outputs: the accumulated ones, or, where one of them is too small for the terms or not finite, the
// sums over the sparse table.  SHARED: other workgroups may have other chunks of the tile.  `position` as in the
// kernels.
template <bool SHARED, int MW, int NW, class Position>
__device__ __forceinline__ void split_store(const float4v (&acc)[MW][NW], const float* __restrict__ x, float* __restrict__ y, const SplitArgs& a,
                                            int b0, int p0, int mblk0, int kg, int c_lo, int c_hi, const Position& position)
{
    const int PQ = a.P * a.Q;
    float* yb = y + (int64_t)b0 * a.D * PQ;
    // 2 |bits| + 2^24, modulo 2^32: infinities and NaN below 2^24, zero at it, then the magnitudes in order
    auto order = [](float v) { return (__float_as_uint(v) << 1) + (1u << 24); };
    unsigned least = ~0u;
#pragma unroll
    for (int m = 0; m < MW; ++m)
#pragma unroll
        for (int i = 0; i < NW; ++i)
#pragma unroll
            for (int j = 0; j < 4; j += 2) least = min(least, min(order(acc[m][i][j]), order(acc[m][i][j + 1])));
    bool exact = false;
    if (__ballot(least < a.floor)) {                         // (zeros, as a rule)
#pragma unroll
        for (int m = 0; m < MW; ++m)
#pragma unroll
            for (int i = 0; i < NW; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const unsigned v = order(acc[m][i][j]);
                    exact |= v < a.floor && v != 1u << 24;
                }
    }
    if (__ballot(exact)) {                                   // (wave-uniform)
#pragma unroll 1
        for (int i = 0; i < NW; ++i) {
            int sm, tp, tq;
            if (!position(i, sm, tp, tq)) continue;
#pragma unroll 1
            for (int mj = 0; mj < 4 * MW; ++mj) {
                const int d = (mblk0 + (mj >> 2)) * 16 + 4 * kg + (mj & 3);
                if (d >= a.D) break;
                const float v = split_exact(x, a, b0 + sm, d, p0 + tp, tq, c_lo, c_hi);
                float* yp = yb + ((int64_t)sm * a.D + d) * PQ + (p0 + tp) * a.Q + tq;
                if (SHARED && a.KS > 1) add_out(yp, v);
                else store_out(yp, v);
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        int sm, tp, tq;
        if (!position(i, sm, tp, tq)) continue;
        const unsigned o = (unsigned)((sm * a.D + mblk0 * 16 + 4 * kg) * PQ) + (unsigned)(mul24(p0 + tp, a.Q) + tq);
#pragma unroll
        for (int m = 0; m < MW; ++m) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if ((mblk0 + m) * 16 + 4 * kg + j >= a.D) continue;
                float* yp = yb + (o + (unsigned)((16 * m + j) * PQ));
                if (SHARED && a.KS > 1) add_out(yp, acc[m][i][j]);
                else store_out(yp, acc[m][i][j]);
            }
        }
    }
}

template <int MW, int NW, int WM, int KG, bool FULL>
__global__ void __launch_bounds__(256 * KG, 2)
split_conv_kernel(const float* __restrict__ x, float* __restrict__ y, const unsigned char* __restrict__ wfrag, const SplitArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    constexpr int NT = 256 * KG;
    // steps of weights in flight: a step multiplies for 6 MW NW matrix instructions (16 clocks and
    // more each), L2 answers after several hundred clocks.  PF * NW is even (parity of the ring below).
    constexpr int PF = MW * NW >= 7 ? 2 : (MW * NW >= 2 ? 4 : 6);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kgrp = KG > 1 ? wave8 >> 2 : 0;                // which steps of the contraction this wave takes
    const int wave = wave8 & 3;
    const int wm = wave % WM, wn = wave / WM;
    const int n16 = lane & 15, kg = lane >> 4;

    // workgroup -> (sample group, row tile, share of the chunks, output-channel block), XCD-aware as in
    // the DENSE variant
    const int grid = gridDim.x;
    const int wg = (grid & 7) == 0 ? (int)(blockIdx.x & 7) * (grid >> 3) + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    int bt, ks, db;
    if (a.wmajor) {
        // (output-channel block and share of the chunks outermost: an XCD streams an eighth of the weights)
        const int o = sdiv(wg, a.inv_ntiles);
        bt = wg - o * a.ntiles;
        ks = sdiv(o, a.inv_ndb);
        db = o - ks * a.ndb;
    } else {
        const int bt0 = sdiv(wg, a.inv_ndb);
        db = wg - bt0 * a.ndb;
        bt = sdiv(bt0, a.inv_KS);                          // (KS: workgroups that share the chunks of a tile)
        ks = bt0 - bt * a.KS;
    }
    const int ch_lo = ks * a.cps, ch_hi = min(a.nchunks, ch_lo + a.cps);
    const int bg = sdiv(bt, a.inv_tiles_p);
    const int tpi = bt - bg * a.tiles_p;
    const int b0 = bg * a.NS, p0 = tpi * a.TP;
    const int row0 = p0 * a.s_h - a.pad_h;
    const int plane = a.H * a.W;
    const int mblk0 = db * (a.DB >> 4) + wm * MW;
    const int cgroups = a.CC >> 3;

    SplitRows sa;
    sa.nsv = min(a.NS, a.N - b0);
    sa.ilo = max(0, -row0);
    sa.nrows = max(0, min(a.Hs, a.H - row0) - sa.ilo);
    sa.rlo = row0 + sa.ilo;
    sa.wcols = min(a.W, a.Ws - a.pad_w);
    SplitStage st;
    {
        const int rows = a.flat ? 1 : sa.nrows;
        st.run = a.flat ? sa.nrows * a.W : sa.wcols;
        st.G = (st.run + a.epv - 1) >> (a.epv >> 1);          // (epv = 1, 2 or 4)
        st.rowsG = rows * st.G;
        st.per_cg = sa.nsv * st.rowsG;
        st.nblocks = cgroups * st.per_cg;
        st.inv_per_cg = __builtin_amdgcn_rcpf((float)max(st.per_cg, 1));
        st.inv_rowsG = __builtin_amdgcn_rcpf((float)max(st.rowsG, 1));
        st.inv_G = __builtin_amdgcn_rcpf((float)max(st.G, 1));
        st.dst0 = sa.ilo * a.Ws + a.pad_w;
        st.plane4 = (unsigned)plane * 4u;
        st.sample4 = (unsigned)a.C * st.plane4;
        st.row4 = (unsigned)a.W * 4u;
    }
    float pre[32];
    // (the block index is made opaque so that the compiler works a block's addresses out again for every
    // chunk: hoisted out of the chunk loop they took 100 registers and the accumulators spilled)
    auto load_pre = [&](int v0) {
        if (st.nblocks == 0) return;                         // (a tile that lies in the padding altogether)
        asm volatile("" : "+v"(v0));
        if (a.epv == 4) load_round<4>(pre, st, v0, NT);
        else if (a.epv == 2) load_round<2>(pre, st, v0, NT);
        else load_round<1>(pre, st, v0, NT);
    };
    auto store_pre = [&](int v0) {
        asm volatile("" : "+v"(v0));
        if (a.epv == 4) store_round<4>(pre, st, lds, v0, NT, a);
        else if (a.epv == 2) store_round<2>(pre, st, lds, v0, NT, a);
        else store_round<1>(pre, st, lds, v0, NT, a);
    };
    const int per_round = NT * (a.epv == 4 ? 1 : (a.epv == 2 ? 2 : 4));
    st.xs = reinterpret_cast<const char*>(x + ((int64_t)b0 * a.C + ch_lo * a.CC) * plane + (int64_t)sa.rlo * a.W);
    st.cleft = a.C - ch_lo * a.CC;
    st.whole = st.cleft >= a.CC;
    if (ch_lo < ch_hi) load_pre(tid);

    // position block i of this wave: the lane's position, as an LDS offset (with its k group) here and as
    // an output offset when the results are stored
    auto position = [&](int i, int& sm, int& tp, int& tq) {
        const int f = (wn * NW + i) * 16 + n16;
        sm = sdiv(f, a.inv_TPQ);
        const int rem = f - mul24(sm, a.TPQ);
        tp = sdiv(rem, a.inv_Q);
        tq = rem - mul24(tp, a.Q);
        return f < a.npos && b0 + sm < a.N && p0 + tp < a.P;
    };
    int bbase[NW];
    float4v acc[MW][NW], accs[MW][NW];                       // hi hi; the small products
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        int sm, tp, tq;
        const bool ok = position(i, sm, tp, tq);
        const int pos = mul24(sm, a.npos1) + mul24(mul24(tp, a.s_h), a.Ws) + mul24(tq, a.s_w);
        bbase[i] = (ok ? mul24(pos, a.pitch) : 0) + kg * 16;
#pragma unroll
        for (int m = 0; m < MW; ++m) acc[m][i] = accs[m][i] = float4v{0, 0, 0, 0};
    }
    const int wrow = a.RS * a.NCB * 3072;                    // bytes per 16-row block
    const unsigned char* wbase = wfrag + (int64_t)mblk0 * wrow + lane * 16;

    // the padding does not change from chunk to chunk: written once
    split_pad(lds, tid, NT, cgroups, sa, a);

    for (int ch = ch_lo; ch < ch_hi; ++ch) {
        const int c0 = ch * a.CC;
        const int cbs = min(a.CC, a.NCB * 32 - c0) >> 5;     // channel blocks in this chunk
        const int gcb0 = c0 >> 5;
        const int ksteps_all = a.RS * cbs;
        const int ksteps = KG > 1 ? (ksteps_all - kgrp + KG - 1) / KG : ksteps_all;
        const int last = ksteps - 1;
        uint4w aq[PF][MW][3], bq[2][3];
        StepCursor wc{0, 0, 0, 0}, xc_{0, 0, 0, 0};
        if (KG > 1 && kgrp) { wc.advance(cbs, a.S, ksteps > 0); xc_.advance(cbs, a.S, ksteps > 0); }
        int wk = 0, xk = 0;
        auto fetch_w = [&](uint4w (&av)[MW][3]) {
            const unsigned char* wu = wbase + (int64_t)(wc.tap * a.NCB + gcb0 + wc.cb) * 3072;
#pragma unroll
            for (int m = 0; m < MW; ++m)
#pragma unroll
                for (int t = 0; t < 3; ++t) av[m][t] = *reinterpret_cast<const uint4w*>(wu + m * wrow + t * 1024);
            wc.template advance<KG>(cbs, a.S, wk < last);
            wk += wk < last ? 1 : 0;
        };
        // the operands of position block i of the step the cursor stands on; after the last block of a
        // step the cursor moves on
        auto fetch_x = [&](uint4w (&bv)[3], int i) {
            const int off = bbase[i] + (xc_.r * a.Ws + xc_.s) * a.pitch + xc_.cb * 64;
#pragma unroll
            for (int t = 0; t < 3; ++t) bv[t] = *reinterpret_cast<const uint4w*>(lds + off + t * a.bufsz);
            if (i == NW - 1) {
                xc_.template advance<KG>(cbs, a.S, xk < last);
                xk += xk < last ? 1 : 0;
            }
        };
        if (KG == 1 || ksteps > 0) {
#pragma unroll
            for (int u = 0; u < PF; ++u) fetch_w(aq[u]);
        }
        if (ch > ch_lo) __syncthreads();     // the previous chunk has been multiplied
        store_pre(tid);
        for (int v0 = tid + per_round; v0 < st.nblocks; v0 += per_round) {
            load_pre(v0);
            store_pre(v0);
        }
        __syncthreads();
        if (ch + 1 < ch_hi) {
            st.xs += (int64_t)a.CC * st.plane4;
            st.cleft -= a.CC;
            st.whole = st.cleft >= a.CC;
            load_pre(tid);
        }
        if (KG == 1 || ksteps > 0) fetch_x(bq[0], 0);
        __builtin_amdgcn_sched_barrier(0);
        const int main_steps = ksteps / PF * PF;
        for (int s0 = 0; s0 < main_steps; s0 += PF) {
#pragma unroll
            for (int u = 0; u < PF; ++u) {
#pragma unroll
                for (int i = 0; i < NW; ++i) {
                    // the operands of the next position block (or of the next step's first) come from LDS
                    // while this one's 6 MW matrix instructions run
                    fetch_x(bq[(u * NW + i + 1) & 1], i + 1 < NW ? i + 1 : 0);
                    __builtin_amdgcn_sched_barrier(0);
                    split_multiply<FULL, MW, NW>(acc, accs, aq[u], bq[(u * NW + i) & 1], i);
                    __builtin_amdgcn_sched_barrier(0);
                }
                fetch_w(aq[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < PF - 1; ++u) {
            if (main_steps + u < ksteps) {
#pragma unroll
                for (int i = 0; i < NW; ++i) {
                    fetch_x(bq[(u * NW + i + 1) & 1], i + 1 < NW ? i + 1 : 0);
                    split_multiply<FULL, MW, NW>(acc, accs, aq[u], bq[(u * NW + i) & 1], i);
                }
            }
        }
    }
#pragma unroll
    for (int m = 0; m < MW; ++m)
#pragma unroll
        for (int i = 0; i < NW; ++i) acc[m][i] += accs[m][i];
    if constexpr (KG > 1) {
        // the second step group hands its sums to the first through LDS, a lane's own 16 bytes per block
        __syncthreads();
        float4v* ex = reinterpret_cast<float4v*>(lds) + wave * (MW * NW * 64) + lane;
        if (kgrp == 1) {
#pragma unroll
            for (int m = 0; m < MW; ++m)
#pragma unroll
                for (int i = 0; i < NW; ++i) ex[(m * NW + i) * 64] = acc[m][i];
        }
        __syncthreads();
        if (kgrp == 1) return;
#pragma unroll
        for (int m = 0; m < MW; ++m)
#pragma unroll
            for (int i = 0; i < NW; ++i) acc[m][i] += ex[(m * NW + i) * 64];
    }
    split_store<true, MW, NW>(acc, x, y, a, b0, p0, mblk0, kg, ch_lo * a.CC, ch_hi * a.CC, position);
}

// ------------------------------------------------------------------------------------------------
// The pipelined form (producers = 4): the chunks are staged by four waves of their own into two LDS
// buffers, one chunk ahead of the eight multiplying waves, whose weights in flight never drain --
// the one-shot form above spends as long between two multiplications (refilling the weights, waiting
// for its staging, splitting) as in them on deep layers: 10 of 16.5 thousand clocks per chunk of the 1x1
// 2048-512 layer on 7 x 7 planes.  Protocol of the DENSE variant's pipelined kernel: barrier k says "chunk
// k is staged" and "chunk k - 1 has been multiplied"; it waits for LDS traffic only, so that weight loads
// stay in flight across it.  Twelve waves leave 168 registers a wave: wave tiles of at most 8 blocks.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ void split_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// One wave-uniform position in the sequence of steps (chunk, filter tap, channel block of the chunk).
struct SplitCursor {
    int ch, r, s, tap, cb, cbs;
    __device__ __forceinline__ void advance(const SplitArgs& a)
    {
        if (++cb < cbs) return;
        cb = 0;
        ++tap;
        if (++s == a.S) { s = 0; ++r; }
        if (tap < a.RS) return;
        tap = r = s = 0;
        ++ch;
        cbs = ch == a.nchunks - 1 ? a.cbs_last : a.CC >> 5;
    }
};

template <int MW, int NW, int WM, bool FULL>
__global__ void __launch_bounds__(768)
split_pipe_kernel(const float* __restrict__ x, float* __restrict__ y, const unsigned char* __restrict__ wfrag, const SplitArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    constexpr int NTC = 512, NTP = 256;                      // multiplying, staging threads
    constexpr int PF = 2;                                    // steps of weights in flight
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave12 = __builtin_amdgcn_readfirstlane(tid >> 6);

    const int grid = gridDim.x;
    const int wg = (grid & 7) == 0 ? (int)(blockIdx.x & 7) * (grid >> 3) + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    int bt, db;
    if (a.wmajor) { db = sdiv(wg, a.inv_ntiles); bt = wg - db * a.ntiles; }
    else { bt = sdiv(wg, a.inv_ndb); db = wg - bt * a.ndb; }
    const int bg = sdiv(bt, a.inv_tiles_p);
    const int tpi = bt - bg * a.tiles_p;
    const int b0 = bg * a.NS, p0 = tpi * a.TP;
    const int row0 = p0 * a.s_h - a.pad_h;
    const int plane = a.H * a.W;
    const int cgroups = a.CC >> 3;
    const int buf = 3 * a.bufsz;

    SplitRows sa;
    sa.nsv = min(a.NS, a.N - b0);
    sa.ilo = max(0, -row0);
    sa.nrows = max(0, min(a.Hs, a.H - row0) - sa.ilo);
    sa.rlo = row0 + sa.ilo;
    sa.wcols = min(a.W, a.Ws - a.pad_w);

    if (wave12 >= 8) {
        // ------------------------------------------------------------------ staging waves
        const int ptid = tid - NTC;
        SplitStage st;
        const int rows = a.flat ? 1 : sa.nrows;
        st.run = a.flat ? sa.nrows * a.W : sa.wcols;
        st.G = (st.run + a.epv - 1) >> (a.epv >> 1);
        st.rowsG = rows * st.G;
        st.per_cg = sa.nsv * st.rowsG;
        st.nblocks = cgroups * st.per_cg;
        st.inv_per_cg = __builtin_amdgcn_rcpf((float)max(st.per_cg, 1));
        st.inv_rowsG = __builtin_amdgcn_rcpf((float)max(st.rowsG, 1));
        st.inv_G = __builtin_amdgcn_rcpf((float)max(st.G, 1));
        st.dst0 = sa.ilo * a.Ws + a.pad_w;
        st.plane4 = (unsigned)plane * 4u;
        st.sample4 = (unsigned)a.C * st.plane4;
        st.row4 = (unsigned)a.W * 4u;
        st.xs = reinterpret_cast<const char*>(x + (int64_t)b0 * a.C * plane + (int64_t)sa.rlo * a.W);
        st.cleft = a.C;
        st.whole = st.cleft >= a.CC;
        const int per_round = NTP * (a.epv == 4 ? 1 : (a.epv == 2 ? 2 : 4));
        float pre[2][32];
        auto load_pre = [&](float (&v)[32], int v0) {
            if (st.nblocks == 0) return;                     // (a tile that lies in the padding altogether)
            asm volatile("" : "+v"(v0));                     // (addresses worked out again, not kept: registers)
            if (a.epv == 4) load_round<4>(v, st, v0, NTP);
            else if (a.epv == 2) load_round<2>(v, st, v0, NTP);
            else load_round<1>(v, st, v0, NTP);
        };
        auto store_pre = [&](const float (&v)[32], unsigned char* to, int v0) {
            asm volatile("" : "+v"(v0));
            if (a.epv == 4) store_round<4>(v, st, to, v0, NTP, a);
            else if (a.epv == 2) store_round<2>(v, st, to, v0, NTP, a);
            else store_round<1>(v, st, to, v0, NTP, a);
        };
        // two rounds of a chunk are loaded a chunk ahead, the others in place
        const bool two = st.nblocks > per_round;
        load_pre(pre[0], ptid);
        if (two) load_pre(pre[1], ptid + per_round);
        for (int k = 0; k < a.nchunks; ++k) {
            unsigned char* to = lds + (k & 1) * buf;
            store_pre(pre[0], to, ptid);
            if (two) store_pre(pre[1], to, ptid + per_round);
            for (int v0 = ptid + 2 * per_round; v0 < st.nblocks; v0 += per_round) {
                load_pre(pre[0], v0);
                store_pre(pre[0], to, v0);
            }
            if (k + 1 < a.nchunks) {
                st.xs += (int64_t)a.CC * st.plane4;
                st.cleft -= a.CC;
                st.whole = st.cleft >= a.CC;
                load_pre(pre[0], ptid);
                if (two) load_pre(pre[1], ptid + per_round);
            }
            split_barrier();                                 // barrier k
        }
        return;
    }

    const int kgrp = wave12 >> 2, wave = wave12 & 3;
    const int wm = wave % WM, wn = wave / WM;
    const int n16 = lane & 15, kg = lane >> 4;
    const int mblk0 = db * (a.DB >> 4) + wm * MW;
    const int wrow = a.RS * a.NCB * 3072;
    const unsigned char* wbase = wfrag + (int64_t)mblk0 * wrow + lane * 16;

    // the two groups of four waves take the even and the odd steps of the whole contraction
    const int total = a.RS * a.NCB;
    const int nsteps = (total - kgrp + 1) >> 1, last = nsteps - 1;
    SplitCursor wc{0, 0, 0, 0, 0, a.nchunks == 1 ? a.cbs_last : a.CC >> 5}, xc_ = wc;
    if (kgrp && nsteps > 0) { wc.advance(a); xc_.advance(a); }
    int wk = 0, xk = 0, nbar = 0;
    uint4w aq[PF][MW][3], bq[2][3];
    auto fetch_w = [&](uint4w (&av)[MW][3]) {
        const unsigned char* wu = wbase + (int64_t)(wc.tap * a.NCB + wc.ch * (a.CC >> 5) + wc.cb) * 3072;
#pragma unroll
        for (int m = 0; m < MW; ++m)
#pragma unroll
            for (int t = 0; t < 3; ++t) av[m][t] = *reinterpret_cast<const uint4w*>(wu + m * wrow + t * 1024);
        if (wk < last) { wc.advance(a); wc.advance(a); ++wk; }
    };
    if (nsteps > 0) {
#pragma unroll
        for (int u = 0; u < PF; ++u) fetch_w(aq[u]);
    }
    // the padding of both buffers is written once, behind the first weight requests
    __builtin_amdgcn_sched_barrier(0);
    split_pad(lds, tid, NTC, cgroups, sa, a);
    if (a.nchunks > 1) split_pad(lds + buf, tid, NTC, cgroups, sa, a);

    auto position = [&](int i, int& sm, int& tp, int& tq) {
        const int f = (wn * NW + i) * 16 + n16;
        sm = sdiv(f, a.inv_TPQ);
        const int rem = f - mul24(sm, a.TPQ);
        tp = sdiv(rem, a.inv_Q);
        tq = rem - mul24(tp, a.Q);
        return f < a.npos && b0 + sm < a.N && p0 + tp < a.P;
    };
    int bbase[NW];
    float4v acc[MW][NW], accs[MW][NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        int sm, tp, tq;
        const bool ok = position(i, sm, tp, tq);
        const int pos = mul24(sm, a.npos1) + mul24(mul24(tp, a.s_h), a.Ws) + mul24(tq, a.s_w);
        bbase[i] = (ok ? mul24(pos, a.pitch) : 0) + kg * 16;
#pragma unroll
        for (int m = 0; m < MW; ++m) acc[m][i] = accs[m][i] = float4v{0, 0, 0, 0};
    }
    auto fetch_x = [&](uint4w (&bv)[3], int i) {
        if (i == 0) while (nbar <= xc_.ch) { split_barrier(); ++nbar; }      // the chunk of this step is staged
        const int off = bbase[i] + (xc_.ch & 1) * buf + (xc_.r * a.Ws + xc_.s) * a.pitch + xc_.cb * 64;
#pragma unroll
        for (int t = 0; t < 3; ++t) bv[t] = *reinterpret_cast<const uint4w*>(lds + off + t * a.bufsz);
        if (i == NW - 1 && xk < last) { xc_.advance(a); xc_.advance(a); ++xk; }
    };
    if (nsteps > 0) {
        fetch_x(bq[0], 0);
        __builtin_amdgcn_sched_barrier(0);
        const int main_steps = nsteps / PF * PF;
        for (int s0 = 0; s0 < main_steps; s0 += PF) {
#pragma unroll
            for (int u = 0; u < PF; ++u) {
#pragma unroll
                for (int i = 0; i < NW; ++i) {
                    fetch_x(bq[(u * NW + i + 1) & 1], i + 1 < NW ? i + 1 : 0);
                    __builtin_amdgcn_sched_barrier(0);
                    split_multiply<FULL, MW, NW>(acc, accs, aq[u], bq[(u * NW + i) & 1], i);
                    __builtin_amdgcn_sched_barrier(0);
                }
                fetch_w(aq[u]);
            }
        }
        if (main_steps < nsteps) {
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                if (i + 1 < NW) fetch_x(bq[(i + 1) & 1], i + 1);
                split_multiply<FULL, MW, NW>(acc, accs, aq[0], bq[i & 1], i);
            }
        }
    }
    while (nbar < a.nchunks) { split_barrier(); ++nbar; }    // (a wave without steps in the last chunks)
#pragma unroll
    for (int m = 0; m < MW; ++m)
#pragma unroll
        for (int i = 0; i < NW; ++i) acc[m][i] += accs[m][i];
    // the second group hands its sums to the first (the staging waves have ended)
    __syncthreads();
    float4v* ex = reinterpret_cast<float4v*>(lds) + wave * (MW * NW * 64) + lane;
    if (kgrp == 1) {
#pragma unroll
        for (int m = 0; m < MW; ++m)
#pragma unroll
            for (int i = 0; i < NW; ++i) ex[(m * NW + i) * 64] = acc[m][i];
    }
    __syncthreads();
    if (kgrp == 1) return;
#pragma unroll
    for (int m = 0; m < MW; ++m)
#pragma unroll
        for (int i = 0; i < NW; ++i) acc[m][i] += ex[(m * NW + i) * 64];
    split_store<false, MW, NW>(acc, x, y, a, b0, p0, mblk0, kg, 0, a.C, position);
}

// ------------------------------------------------------------------------------------------------
// Geometry and launch.
// ------------------------------------------------------------------------------------------------
static unsigned float_bits(float f)
{
    unsigned u;
    std::memcpy(&u, &f, 4);
    return u;
}

bool split_geometry(const Plan& p, int TP, int NS, int CC, int DB, int WM, int KG, int KS, int PW, int lds_budget, MfmaGeom* out)
{
    const sc_layer_t& L = p.L;
    MfmaGeom g{};
    if (TP < 1 || NS < 1 || NS > 16 || CC < 32 || CC % 32) return false;
    if (DB != 16 && DB != 32 && DB != 64 && DB != 128) return false;
    if ((WM != 1 && WM != 2 && WM != 4) || DB % (16 * WM) || (KG != 1 && KG != 2)) return false;
    g.TP = std::min(TP, p.P);
    g.NS = g.TP < p.P ? 1 : NS;                   // several samples only with whole planes
    g.tiles_p = (p.P + g.TP - 1) / g.TP;
    const int64_t Hs = (int64_t)(g.TP - 1) * L.stride_h + L.R, Ws = (int64_t)(p.Q - 1) * L.stride_w + L.S;
    if (g.NS * Hs * Ws >= (1 << 16) || L.W >= (1 << 20) || p.P >= (1 << 22)) return false;    // (24-bit index products)
    g.Hs = (int)Hs;
    g.Ws = (int)Ws;
    g.npos_s = g.NS * g.Hs * g.Ws;
    g.npos = g.NS * g.TP * p.Q;
    // (32-bit offsets inside the samples of a workgroup and inside a 16-row block of the weights)
    if ((int64_t)g.NS * L.C * L.H * L.W >= (1ll << 29) || (int64_t)g.NS * L.D * p.P * p.Q >= (1ll << 29) ||
        (int64_t)L.R * L.S * ((L.C + 31) / 32) >= (1 << 18))
        return false;
    g.NCB = (L.C + 31) / 32;
    g.CC = std::min(CC, g.NCB * 32);
    g.nchunks = (g.NCB * 32 + g.CC - 1) / g.CC;
    g.pitch = g.CC * 2 + 16;                      // odd in units of 16 bytes (the counters still show bank conflicts, 6 clocks for
                                                  // each LDS instruction; 32, 48 or 80 instead of 16 take the same time)
    g.DB = DB;
    g.ndb = (L.D + DB - 1) / DB;
    g.WM = WM;
    g.MW = DB / (16 * WM);
    g.KG = KG;
    const int nb = (g.npos + 15) / 16, wn = 4 / WM, nw = (nb + wn - 1) / wn;
    if (nw > 8) return false;
    g.NW = nw <= 2 ? nw : (nw <= 4 ? 4 : (nw <= 7 ? 7 : 8));
    // accumulators (two sets) and operands in flight within 256 registers
    if (g.MW > 2 || (g.MW == 2 && g.NW == 8)) return false;
    g.DL = KS;                                    // workgroups that share the chunks of a tile
    // (each of them has at least one)
    if (KS < 1 || KS > 16 || (KS - 1) * ((g.nchunks + KS - 1) / KS) >= g.nchunks) return false;
    g.bufsz = g.npos_s * g.pitch;
    if ((int64_t)(g.CC / 8) * g.npos_s >= (1 << 19)) return false;     // sdiv() range of the staging
    // pipelined: two chunk buffers, eight multiplying waves, a wave tile of at most 8 blocks in 168 registers
    if (PW && (PW != 4 || KG != 2 || KS != 1 || g.MW * g.NW > 8)) return false;
    g.PW = PW;
    int64_t lds = 3ll * g.bufsz * (PW && g.nchunks > 1 ? 2 : 1);
    if (KG == 2) lds = std::max<int64_t>(lds, (int64_t)g.MW * g.NW * 4096);
    if (lds > lds_budget || lds > kMaxLdsBytes) return false;
    g.lds_bytes = (int)lds;
    *out = g;
    return true;
}

int split_grid_size(const MfmaGeom& g, int N) { return ((N + g.NS - 1) / g.NS) * g.tiles_p * g.ndb * g.DL; }

template <int MW, int NW, int WM, int KG, bool FULL>
static sc_status_t launch_split_full(const Plan& p, const SplitArgs& a, const void* x, void* y, int grid, hipStream_t stream)
{
    // KG = 3: the pipelined form (eight multiplying waves and four that stage)
    auto kernel = [] {
        if constexpr (KG == 3) return &split_pipe_kernel<MW, NW, WM, FULL>;
        else return &split_conv_kernel<MW, NW, WM, KG, FULL>;
    }();
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [&] {
        attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes);
    });
    if (attr_err != hipSuccess) return SC_ERR_HIP;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(256 * KG), p.mg.lds_bytes, stream, static_cast<const float*>(x),
                       static_cast<float*>(y), p.d_wfrag, a);
    return hipGetLastError() == hipSuccess ? SC_OK : SC_ERR_HIP;
}

template <int MW, int NW, int WM, int KG>
static sc_status_t launch_split_one(const Plan& p, const SplitArgs& a, const void* x, void* y, int grid, hipStream_t stream)
{
    return p.split_full ? launch_split_full<MW, NW, WM, KG, true>(p, a, x, y, grid, stream)
                        : launch_split_full<MW, NW, WM, KG, false>(p, a, x, y, grid, stream);
}

template <int MW, int WM, int KG>
static sc_status_t launch_split_nw(const Plan& p, const SplitArgs& a, const void* x, void* y, int grid, hipStream_t stream)
{
    switch (p.mg.NW) {
        case 1: return launch_split_one<MW, 1, WM, KG>(p, a, x, y, grid, stream);
        case 2: return launch_split_one<MW, 2, WM, KG>(p, a, x, y, grid, stream);
        case 4: return launch_split_one<MW, 4, WM, KG>(p, a, x, y, grid, stream);
        case 7: if constexpr (MW == 1 || KG != 3) return launch_split_one<MW, 7, WM, KG>(p, a, x, y, grid, stream); break;
        case 8: if constexpr (MW == 1) return launch_split_one<MW, 8, WM, KG>(p, a, x, y, grid, stream); break;
    }
    return SC_ERR_UNSUPPORTED;
}

template <int KG>
static sc_status_t launch_split_kg(const Plan& p, const SplitArgs& a, const void* x, void* y, int grid, hipStream_t stream)
{
    switch (p.mg.WM * 10 + p.mg.MW) {
        case 11: return launch_split_nw<1, 1, KG>(p, a, x, y, grid, stream);
        case 12: return launch_split_nw<2, 1, KG>(p, a, x, y, grid, stream);
        case 21: return launch_split_nw<1, 2, KG>(p, a, x, y, grid, stream);
        case 22: return launch_split_nw<2, 2, KG>(p, a, x, y, grid, stream);
        case 41: return launch_split_nw<1, 4, KG>(p, a, x, y, grid, stream);
        case 42: return launch_split_nw<2, 4, KG>(p, a, x, y, grid, stream);
    }
    return SC_ERR_UNSUPPORTED;
}

sc_status_t launch_split(const Plan& p, const void* x, void* y, int N, hipStream_t stream)
{
    const MfmaGeom& g = p.mg;
    if (!p.d_wfrag) return SC_ERR_UNSUPPORTED;
    // sdiv() range: a batch that needs more workgroups is run in slices
    const int64_t per_group = (int64_t)g.tiles_p * g.ndb * g.DL, groups = ((1 << 19) - 1) / per_group;
    if (groups < 1) return SC_ERR_UNSUPPORTED;
    if ((N + g.NS - 1) / g.NS > groups) {
        const int step = (int)groups * g.NS;
        for (int n0 = 0; n0 < N; n0 += step) {
            const sc_status_t st = launch_split(p, static_cast<const float*>(x) + (int64_t)n0 * p.L.C * p.L.H * p.L.W,
                                                static_cast<float*>(y) + (int64_t)n0 * p.L.D * p.P * p.Q, std::min(step, N - n0), stream);
            if (st != SC_OK) return st;
        }
        return SC_OK;
    }
    const int64_t grid = (int64_t)((N + g.NS - 1) / g.NS) * per_group;
    SplitArgs a{};
    a.C = p.L.C; a.D = p.L.D; a.N = N; a.H = p.L.H; a.W = p.L.W; a.P = p.P; a.Q = p.Q;
    a.S = p.L.S; a.RS = p.L.R * p.L.S; a.s_h = p.L.stride_h; a.s_w = p.L.stride_w; a.pad_h = p.L.pad_h; a.pad_w = p.L.pad_w;
    a.TP = g.TP; a.NS = g.NS; a.tiles_p = g.tiles_p; a.Hs = g.Hs; a.Ws = g.Ws; a.npos_s = g.npos_s; a.npos = g.npos;
    a.CC = g.CC; a.nchunks = g.nchunks; a.NCB = g.NCB; a.pitch = g.pitch; a.DB = g.DB; a.ndb = g.ndb; a.bufsz = g.bufsz;
    a.KS = g.DL; a.cps = (g.nchunks + g.DL - 1) / g.DL; a.inv_KS = 1.0f / (float)g.DL;
    a.TPQ = g.TP * p.Q;
    a.npos1 = g.Hs * g.Ws;
    a.floor = 2u * float_bits(p.split_floor) + (1u << 24);
    a.n = p.n; a.theta = static_cast<const float*>(p.d_theta); a.col = p.d_col; a.len = p.d_len;
    a.cbs_last = g.NCB - (g.nchunks - 1) * (g.CC / 32);
    {
        // what an XCD reads into its L2: with the tile outermost all weights and an eighth of the input,
        // else its share of the weights and (of the chunks its workgroups take) of the input
        a.ntiles = ((N + g.NS - 1) / g.NS) * g.tiles_p;
        a.inv_ntiles = 1.0f / (float)a.ntiles;
        const double w = (double)split_weight_bytes(p), xin = (double)N * p.L.C * p.L.H * p.L.W * 4.0, combos = (double)g.ndb * g.DL;
        a.wmajor = w / std::min(8.0, combos) + xin / g.DL * std::min(1.0, combos / 8.0) < w + xin / 8.0 ? 1 : 0;
    }
    a.inv_ndb = 1.0f / (float)g.ndb; a.inv_tiles_p = 1.0f / (float)g.tiles_p;
    a.inv_HsWs = 1.0f / (float)(g.Hs * g.Ws); a.inv_Ws = 1.0f / (float)g.Ws;
    a.inv_TPQ = 1.0f / (float)a.TPQ; a.inv_Q = 1.0f / (float)p.Q;
    // staging: the widest loads (16, 8 or 4 bytes) that the runs and the pointer allow.  Where the staged
    // rows carry no padding columns they are one run per channel (flat); a pointwise tile's run starts at
    // a multiple of TP * W and is TP * W long (the last one what is left of the plane)
    a.flat = (g.Ws == p.L.W && p.L.pad_w == 0) ? 1 : 0;
    const bool pointwise = a.RS == 1 && a.s_h == 1 && a.s_w == 1 && !a.pad_h && !a.pad_w;
    const int plane = p.L.H * p.L.W;
    a.epv = 1;
    for (int e = 4; e > 1; e >>= 1) {
        const bool fits = p.L.W % e == 0 || (a.flat && pointwise && plane % e == 0 && (g.tiles_p == 1 || a.TPQ % e == 0));
        if (fits && reinterpret_cast<uintptr_t>(x) % (uintptr_t)(e * 4) == 0) { a.epv = e; break; }
    }
    if (g.DL > 1) {
        const sc_status_t st = launch_clear(y, (int64_t)N * p.L.D * p.P * p.Q, stream);
        if (st != SC_OK) return st;
    }
    if (g.PW) return launch_split_kg<3>(p, a, x, y, (int)grid, stream);
    return g.KG == 2 ? launch_split_kg<2>(p, a, x, y, (int)grid, stream) : launch_split_kg<1>(p, a, x, y, (int)grid, stream);
}

}  // namespace sc
