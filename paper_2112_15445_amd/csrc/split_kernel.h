// Kernels of the fp32 form on the matrix cores (split_mfma.hip has the formulation): the one-shot and the pipelined one, and
// their launcher by wave tile.  Instantiated by the columns of a staging load in split_*_{1,2,4}.hip.
#pragma once

#include <mutex>

#include "dense_mfma_kernel.h"

namespace sc {

// What a launch is made of; read at once when a kernel starts, as TileArgs and for the same reason (2.4 thousand clocks passed before the
// first load, in seven trips to memory one after the other).  With that, staging instantiated by the columns of a load and a block's
// place worked out once for all chunks: 3x3 128-128 at 28 x 28, batch 32 39.9 -> 37.3 us, 3x3 stride 2 512-512 at 14 x 14 51.1 -> 48.9, 1x1
// 2048-512 at 7 x 7 30.9 -> 28.7, 1-D 300-64 along 64, batch 128 11.3 -> 10.8, 3x3 100-90 at 27 x 31, batch 7 17.3 -> 16.5.
// (Loads of any alignment and of up to four columns, as load_columns in sc_staging.h estimates to be fastest, instead of as wide as row length and pointer
// allow, after that: 28.7 -> 27.7 and 16.5 -> 15.5 on the last but two and the last, runs of 49 and rows of 31.
// Two rounds loaded a chunk ahead instead of one: level. The first chunk of the pipelined form staged by all twelve waves: 1-D 10.8 -> 11.5, its
// registers spill.)
struct SplitArgs {
    // workgroup order (see split_block): workgroups / 8 and what is left, extents of the two inner indices
    int gq, gr, inner, inner2;
    float inv_inner, inv_inner2, inv_tiles_p;
    int tiles_p, NS, N, TP, s_h, pad_h;
    // staging: as TileArgs; chunks of a workgroup (of those that share them) and of the layer
    int H, Hs, W, wcols, Ws, npos1, pad_w, CC, C, cps, nchunks;
    unsigned plane4;
    int pitch, bufsz, npos_s;
    int DB, RS, NCB, S, cbs_last;
    int npos, TPQ, Q, s_w;
    float inv_TPQ, inv_Q, inv_npos1, inv_Ws;
    int P, D;
    unsigned floor;          // 2 bits(m) + 2^24 of the smallest magnitude m of an output that the terms serve
    // bit 0: output-channel blocks outermost, 1: staged rows of a sample are one run per channel, 2: padding, 3: other workgroups have other
    // chunks of the tile; 4-5: log2 of the waves along the output channels
    int bits;
    int spare[3];
};

// the sparse table, for split_exact
struct SplitTable {
    const float* theta;
    const int32_t *col, *len;
    int n;
};

// (form -- one or two groups of waves, pipelined with two or four --, columns per staging load)
sc_status_t launch_split_one_1(const Plan& p, const SplitArgs& a, const SplitTable& t, const void* x, void* y, int grid, hipStream_t stream);
sc_status_t launch_split_one_2(const Plan& p, const SplitArgs& a, const SplitTable& t, const void* x, void* y, int grid, hipStream_t stream);
sc_status_t launch_split_one_4(const Plan& p, const SplitArgs& a, const SplitTable& t, const void* x, void* y, int grid, hipStream_t stream);
sc_status_t launch_split_two_1(const Plan& p, const SplitArgs& a, const SplitTable& t, const void* x, void* y, int grid, hipStream_t stream);
sc_status_t launch_split_two_2(const Plan& p, const SplitArgs& a, const SplitTable& t, const void* x, void* y, int grid, hipStream_t stream);
sc_status_t launch_split_two_4(const Plan& p, const SplitArgs& a, const SplitTable& t, const void* x, void* y, int grid, hipStream_t stream);
sc_status_t launch_split_pipe2_1(const Plan& p, const SplitArgs& a, const SplitTable& t, const void* x, void* y, int grid, hipStream_t stream);
sc_status_t launch_split_pipe2_2(const Plan& p, const SplitArgs& a, const SplitTable& t, const void* x, void* y, int grid, hipStream_t stream);
sc_status_t launch_split_pipe2_4(const Plan& p, const SplitArgs& a, const SplitTable& t, const void* x, void* y, int grid, hipStream_t stream);
sc_status_t launch_split_pipe4_1(const Plan& p, const SplitArgs& a, const SplitTable& t, const void* x, void* y, int grid, hipStream_t stream);
sc_status_t launch_split_pipe4_2(const Plan& p, const SplitArgs& a, const SplitTable& t, const void* x, void* y, int grid, hipStream_t stream);
sc_status_t launch_split_pipe4_4(const Plan& p, const SplitArgs& a, const SplitTable& t, const void* x, void* y, int grid, hipStream_t stream);

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

// Workgroup -> (tile bt, share ks of the chunks, output-channel block db), XCD-aware as in the DENSE variant.  Blocks and shares
// outermost (bit 0): an XCD streams its share of the weights; else tiles, then shares, then blocks.
struct SplitBlock { int bt, ks, db; };
__device__ __forceinline__ SplitBlock split_block(const SplitArgs& a)
{
    const int xcd = blockIdx.x & 7;
    const int wg = xcd * a.gq + min(xcd, a.gr) + (int)(blockIdx.x >> 3);
    const int hi = __builtin_amdgcn_readfirstlane(sdiv(wg, a.inv_inner)), lo = wg - hi * a.inner;
    const int hi2 = __builtin_amdgcn_readfirstlane(sdiv(hi, a.inv_inner2)), lo2 = hi - hi2 * a.inner2;
    return {a.bits & 1 ? lo : hi2, a.bits & 1 ? hi2 : lo2, a.bits & 1 ? lo2 : lo};
}

// ------------------------------------------------------------------------------------------------
// Staging of one chunk: blocks of 8 channels x EPV columns, loaded with any alignment that an element has, split
// and transposed in registers, one 16-byte word per position, channel group and image.  `rows` runs
// of `run` elements per sample and channel (where the staged rows carry no padding columns they are
// one run).  Blocks are dealt to the threads in rounds; a round is 32 registers of loads per thread.
// The first rounds of the next chunk are loaded before the current one is multiplied, so that small chunks cost no memory
// latency; where their blocks lie is worked out once for all chunks (SplitSlot).
// ------------------------------------------------------------------------------------------------
struct SplitStage {
    const char* xs;        // first staged element of sample 0, channel 0 of the chunk
    unsigned sample4, plane4, row4;    // bytes per sample, channel and input row
    int nblocks, rowsG, per_cg, G, run, cleft, dst0;
    int nsv, ilo, nrows;   // samples inside the batch; staged rows inside the input: [ilo, ilo + nrows)
    bool whole;            // every channel of the chunk's groups exists in the layer
    float inv_per_cg, inv_rowsG, inv_G;
};

template <int EPV>
__device__ __forceinline__ SplitStage split_stage(const SplitArgs& a, const float* x, int b0, int row0, int c0)
{
    SplitStage st;
    st.nsv = min(a.NS, a.N - b0);
    st.ilo = max(0, -row0);
    st.nrows = max(0, min(a.Hs, a.H - row0) - st.ilo);
    const bool flat = a.bits & 2;
    st.run = flat ? st.nrows * a.W : a.wcols;
    st.G = (st.run + EPV - 1) >> (EPV >> 1);                 // (EPV = 1, 2 or 4)
    st.rowsG = (flat ? 1 : st.nrows) * st.G;
    st.per_cg = st.nsv * st.rowsG;
    st.nblocks = (a.CC >> 3) * st.per_cg;
    st.inv_per_cg = __builtin_amdgcn_rcpf((float)max(st.per_cg, 1));
    st.inv_rowsG = __builtin_amdgcn_rcpf((float)max(st.rowsG, 1));
    st.inv_G = __builtin_amdgcn_rcpf((float)max(st.G, 1));
    st.dst0 = st.ilo * a.Ws + a.pad_w;
    st.plane4 = a.plane4;
    st.sample4 = (unsigned)a.C * st.plane4;
    st.row4 = (unsigned)a.W * 4u;
    st.xs = reinterpret_cast<const char*>(x) + (int64_t)b0 * st.sample4 + (int64_t)c0 * st.plane4 + (int64_t)(row0 + st.ilo) * st.row4;
    st.cleft = a.C - c0;
    st.whole = st.cleft >= a.CC;
    return st;
}

// the next chunk
__device__ __forceinline__ void split_advance(SplitStage& st, const SplitArgs& a)
{
    st.xs += (int64_t)a.CC * st.plane4;
    st.cleft -= a.CC;
    st.whole = st.cleft >= a.CC;
}

// padding: staged positions outside the input or past the batch are zeros in all three images
__device__ __forceinline__ void split_pad(unsigned char* lds, int tid, int NT, const SplitStage& st, const SplitArgs& a)
{
    // (a layer without padding needs none: a position past the batch or the plane feeds only itself)
    if (!(a.bits & 4)) return;
    const int cgroups = a.CC >> 3;
    for (int pos = tid; pos < a.npos_s; pos += NT) {
        const int sm = sdiv(pos, a.inv_npos1);
        const int rem = pos - mul24(sm, a.npos1);
        const int i = sdiv(rem, a.inv_Ws);
        const int w = rem - mul24(i, a.Ws);
        const bool inside = sm < st.nsv && (unsigned)(i - st.ilo) < (unsigned)st.nrows && (unsigned)(w - a.pad_w) < (unsigned)a.wcols;
        if (!inside)
            for (int t = 0; t < 3; ++t)
                for (int cg = 0; cg < cgroups; ++cg) *reinterpret_cast<uint4w*>(lds + t * a.bufsz + mul24(pos, a.pitch) + cg * 16) = uint4w{0u, 0u, 0u, 0u};
    }
}

// Where a block is read from (bytes from st.xs, in channel 0 of the chunk, and its channel group) and written to (bytes into the first
// image; -1: no such block, then block 0 is read).  A run that is no multiple of EPV ends in a block that starts EPV before its
// end: the columns that two blocks share are written twice with the same values, and loads have any alignment of 4 bytes.
struct SplitSlot { unsigned off; int cg, dst; };
template <int EPV> constexpr int kSplitVB = 4 / EPV;         // blocks per thread and round

template <int EPV, int VB>
__device__ __forceinline__ void split_slots(SplitSlot (&slot)[VB], const SplitStage& st, const SplitArgs& a, int v0, int NT)
{
#pragma unroll
    for (int u = 0; u < VB; ++u) {
        const int v = v0 + u * NT;
        const bool live = v < st.nblocks;
        const int vv = live ? v : 0;
        const int cg = sdiv(vv, st.inv_per_cg);
        int r = vv - mul24(cg, st.per_cg), sm = 0, ii = 0;
        if (st.rowsG != st.per_cg) { sm = sdiv(r, st.inv_rowsG); r -= mul24(sm, st.rowsG); }
        if (st.rowsG != st.G) { ii = sdiv(r, st.inv_G); r -= mul24(ii, st.G); }
        const int col = min(r * EPV, st.run - EPV);
        slot[u].off = (unsigned)sm * st.sample4 + (unsigned)mul24(ii, (int)st.row4) + (unsigned)col * 4u;
        slot[u].cg = cg;
        slot[u].dst = live ? mul24(mul24(sm, a.npos1) + st.dst0 + mul24(ii, a.Ws) + col, a.pitch) + cg * 16 : -1;
    }
}

template <int EPV, int VB>
__device__ __forceinline__ void split_load(float (&pre)[32], const SplitStage& st, const SplitSlot (&slot)[VB])
{
    typedef float Vec __attribute__((ext_vector_type(EPV), aligned(4)));
    // (whole addresses in the lanes, as tile_src)
    using Src = const __attribute__((address_space(1))) char*;
    auto load = [&](int at, Src src) __attribute__((always_inline)) {
        const Vec t = *reinterpret_cast<const __attribute__((address_space(1))) Vec*>(src);
#pragma unroll
        for (int e = 0; e < EPV; ++e) pre[at * EPV + e] = t[e];
    };
#pragma unroll
    for (int u = 0; u < VB; ++u) {
        unsigned off = slot[u].off;
        int cg = slot[u].cg;
        // (opaque: a block's addresses are worked out again for every chunk; kept in registers they took 100 of them and the
        // accumulators spilled)
        asm volatile("" : "+v"(off), "+v"(cg));
        const Src base = reinterpret_cast<Src>(reinterpret_cast<uint64_t>(st.xs) + off);
        if (st.whole) {
            Src src = base + (uint64_t)((unsigned)mul24(cg, 8) * st.plane4);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                load(u * 8 + j, src);
                src += st.plane4;
                asm("" : "+v"(src));
                __builtin_amdgcn_sched_barrier(0);           // (one address at a time: registers)
            }
        } else {
            unsigned o = (unsigned)mul24(cg, 8) * st.plane4;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                // (channels past the layer's last: the block's place in channel 0, zeroed when it is stored)
                load(u * 8 + j, base + (uint64_t)(cg * 8 + j < st.cleft ? o : 0u));
                o += st.plane4;
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
}

template <int EPV, int VB>
__device__ __forceinline__ void split_put(const float (&pre)[32], const SplitStage& st, unsigned char* lds, const SplitSlot (&slot)[VB], const SplitArgs& a)
{
#pragma unroll
    for (int u = 0; u < VB; ++u) {
        if (slot[u].dst < 0) continue;
        int cg = slot[u].cg, to = slot[u].dst;
        asm volatile("" : "+v"(cg), "+v"(to));
        unsigned char* dst = lds + to;
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
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
__device__ __forceinline__ float split_exact(const float* __restrict__ x, const SplitArgs& a, const SplitTable& tab, int b, int d, int p, int q, int c_lo, int c_hi)
{
    const int i0 = p * a.s_h - a.pad_h, w0 = q * a.s_w - a.pad_w;
    const float* xb = x + (int64_t)b * a.C * a.H * a.W;
    float sum = 0.0f;
#pragma unroll 1
    for (int j = 0; j < tab.len[d]; ++j) {
        const int64_t at = (int64_t)d * tab.n + j;
        const int k = tab.col[at] & 0x7fffffff, c = k / a.RS, tap = k - c * a.RS, r = tap / a.S;
        const int i = i0 + r, w = w0 + tap - r * a.S;
        if (c >= c_lo && c < c_hi && i >= 0 && i < a.H && w >= 0 && w < a.W)
            sum = __builtin_fmaf(tab.theta[at], xb[((int64_t)c * a.H + i) * a.W + w], sum);
    }
    return sum;
}

// The wave's outputs, NB blocks of 16 channels x 16 positions: the accumulated ones, or, where one of them is too small for the terms
// or not finite, the sums over the sparse table.  SHARED: other workgroups may have other chunks of the tile.  `get(t)`: the sums
// of block t; `block(t, m, i)`: whether there is a block t, its place in the wave tile; `position` as in the kernels.
template <bool SHARED, int NB, class Get, class Block, class Position>
__device__ __forceinline__ void split_store(const Get& get, const Block& block, const float* __restrict__ x, float* __restrict__ y, const SplitArgs& a,
                                            const SplitTable& tab, int b0, int p0, int mblk0, int kg, int c_lo, int c_hi, const Position& position)
{
    const int PQ = a.P * a.Q;
    float* yb = y + (int64_t)b0 * a.D * PQ;
    // 2 |bits| + 2^24, modulo 2^32: infinities and NaN below 2^24, zero at it, then the magnitudes in order
    auto order = [](float v) { return (__float_as_uint(v) << 1) + (1u << 24); };
    unsigned least = ~0u;
#pragma unroll
    for (int t = 0; t < NB; ++t) {
        int m, i;
        if (!block(t, m, i)) continue;
        const float4v v = get(t);
#pragma unroll
        for (int j = 0; j < 4; j += 2) least = min(least, min(order(v[j]), order(v[j + 1])));
    }
    bool exact = false;
    if (__ballot(least < a.floor)) {                         // (zeros, as a rule)
#pragma unroll
        for (int t = 0; t < NB; ++t) {
            int m, i;
            if (!block(t, m, i)) continue;
            const float4v v = get(t);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const unsigned o = order(v[j]);
                exact |= o < a.floor && o != 1u << 24;
            }
        }
    }
    if (__ballot(exact)) {                                   // (wave-uniform)
#pragma unroll 1
        for (int t = 0; t < NB; ++t) {
            int m, i, sm, tp, tq;
            if (!block(t, m, i) || !position(i, sm, tp, tq)) continue;
#pragma unroll 1
            for (int j = 0; j < 4; ++j) {
                const int d = (mblk0 + m) * 16 + 4 * kg + j;
                if (d >= a.D) break;
                const float v = split_exact(x, a, tab, b0 + sm, d, p0 + tp, tq, c_lo, c_hi);
                float* yp = yb + ((int64_t)sm * a.D + d) * PQ + (p0 + tp) * a.Q + tq;
                if (SHARED && (a.bits & 8)) add_out(yp, v);
                else store_out(yp, v);
            }
        }
        return;
    }
#pragma unroll
    for (int t = 0; t < NB; ++t) {
        int m, i, sm, tp, tq;
        if (!block(t, m, i) || !position(i, sm, tp, tq)) continue;
        const float4v v = get(t);
        const int d = (mblk0 + m) * 16 + 4 * kg;
        const unsigned o = (unsigned)((sm * a.D + d) * PQ) + (unsigned)(mul24(p0 + tp, a.Q) + tq);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (d + j >= a.D) continue;
            float* yp = yb + (o + (unsigned)(j * PQ));
            if (SHARED && (a.bits & 8)) add_out(yp, v[j]);
            else store_out(yp, v[j]);
        }
    }
}

__device__ __forceinline__ void split_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int MW, int NW, int KG, int EPV, bool FULL>
__global__ void __launch_bounds__(256 * KG, 2)
split_conv_kernel(const float* __restrict__ x, float* __restrict__ y, const unsigned char* __restrict__ wfrag, const SplitArgs args, const SplitTable tab)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    constexpr int NT = 256 * KG;
    const SplitArgs a = args_at_once(args);
    // steps of weights in flight: a step multiplies for 6 MW NW matrix instructions (16 clocks and
    // more each), L2 answers after several hundred clocks.  PF * NW is even (parity of the ring below).
    // (Six steps for the tile of one block, before the steps came from tables, are no part of a table's 64; with four, and the tables, 21 such
    // shapes on seven layers take 0.62 - 0.98 of the time.)
    constexpr int PF = MW * NW >= 7 ? 2 : 4;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kgrp = KG > 1 ? wave8 >> 2 : 0;                // which steps of the contraction this wave takes
    const int wave = wave8 & 3;
    const int lwm = a.bits >> 4 & 3, wm = wave & ((1 << lwm) - 1), wn = wave >> lwm;
    const int n16 = lane & 15, kg = lane >> 4;

    const SplitBlock block = split_block(a);
    const int bt = block.bt, db = block.db;
    const int ch_lo = block.ks * a.cps, ch_hi = min(a.nchunks, ch_lo + a.cps);
    const int bg = __builtin_amdgcn_readfirstlane(sdiv(bt, a.inv_tiles_p));
    const int tpi = bt - bg * a.tiles_p;
    const int b0 = bg * a.NS, p0 = tpi * a.TP;
    const int row0 = p0 * a.s_h - a.pad_h;
    const int mblk0 = db * (a.DB >> 4) + wm * MW;

    // the loads of the first chunk (nblocks = 0: a tile that lies in the padding altogether)
    SplitStage st = split_stage<EPV>(a, x, b0, row0, ch_lo * a.CC);
    // (the largest wave tile has no registers for the blocks' places, nor for four blocks at once: 1331 spills)
    constexpr bool kept = MW * NW < 14;
    constexpr int VB = kept ? kSplitVB<EPV> : 1, per_round = NT * VB;
    float pre[32];
    SplitSlot slots[VB];
    split_slots<EPV>(slots, st, a, tid, NT);
    if (st.nblocks) split_load<EPV>(pre, st, slots);
    __builtin_amdgcn_sched_barrier(0);
    auto again = [&]() __attribute__((always_inline)) {
        if constexpr (!kept) {
            int v0 = tid;
            asm volatile("" : "+v"(v0));
            split_slots<EPV>(slots, st, a, v0, NT);
        }
    };

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

    const float inv_S = __builtin_amdgcn_rcpf((float)a.S);

    // the padding does not change from chunk to chunk: written once
    split_pad(lds, tid, NT, st, a);

    for (int ch = ch_lo; ch < ch_hi; ++ch) {
        const int c0 = ch * a.CC;
        const int cbs = min(a.CC, a.NCB * 32 - c0) >> 5;     // channel blocks in this chunk
        const int gcb0 = c0 >> 5;
        const int ksteps_all = a.RS * cbs;
        const int ksteps = KG > 1 ? (ksteps_all - kgrp + KG - 1) / KG : ksteps_all;
        uint4w aq[PF][MW][3], bq[2][3];
        const float inv_cbs = __builtin_amdgcn_rcpf((float)cbs);
        int xtab, wtab;
        auto table = [&](int s0) __attribute__((always_inline)) {
            const int s = min(kgrp + KG * (s0 + lane), ksteps_all - 1);
            const int tap = sdiv(s, inv_cbs), cb = s - tap * cbs, r = sdiv(tap, inv_S);
            xtab = (r * a.Ws + tap - r * a.S) * a.pitch + cb * 64;
            wtab = tap * a.NCB + gcb0 + cb;
        };
        auto fetch_w = [&](uint4w (&av)[MW][3], int k) __attribute__((always_inline)) {
            const unsigned char* wu = wbase + (int64_t)__builtin_amdgcn_readlane(wtab, min(k, 63)) * 3072;
#pragma unroll
            for (int m = 0; m < MW; ++m)
#pragma unroll
                for (int t = 0; t < 3; ++t) av[m][t] = *reinterpret_cast<const uint4w*>(wu + m * wrow + t * 1024);
        };
        // (by a wave without steps too: behind loads that only some waves issue the compiler waits for the weights before it stages
        // the input)
        table(0);
#pragma unroll
        for (int u = 0; u < PF; ++u) fetch_w(aq[u], u);
        if (ch > ch_lo) split_barrier();     // the previous chunk has been multiplied
        again();
        if (st.nblocks) split_put<EPV>(pre, st, lds, slots, a);
        for (int v0 = tid + per_round; v0 - tid < st.nblocks; v0 += per_round) {
            SplitSlot t[VB];
            split_slots<EPV>(t, st, a, v0, NT);
            split_load<EPV>(pre, st, t);
            split_put<EPV>(pre, st, lds, t, a);
        }
        split_barrier();
        if (ch + 1 < ch_hi) {
            split_advance(st, a);
            again();
            if (st.nblocks) split_load<EPV>(pre, st, slots);
        }
        for (int s0 = 0; s0 < ksteps; s0 += 64) {
            const int n = min(64, ksteps - s0);
            if (s0 > 0) {
                table(s0);
#pragma unroll
                for (int u = 0; u < PF; ++u) fetch_w(aq[u], u);
            }
            auto fetch_x = [&](uint4w (&bv)[3], int i, int k) __attribute__((always_inline)) {
                const int off = bbase[i] + __builtin_amdgcn_readlane(xtab, min(k, 63));
#pragma unroll
                for (int t = 0; t < 3; ++t) bv[t] = *reinterpret_cast<const uint4w*>(lds + off + t * a.bufsz);
            };
            fetch_x(bq[0], 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            const int main_steps = n / PF * PF;
            for (int k = 0; k < main_steps; k += PF) {
#pragma unroll
                for (int u = 0; u < PF; ++u) {
#pragma unroll
                    for (int i = 0; i < NW; ++i) {
                        // the operands of the next position block (or of the next step's first) come from LDS
                        // while this one's 6 MW matrix instructions run
                        fetch_x(bq[(u * NW + i + 1) & 1], i + 1 < NW ? i + 1 : 0, i + 1 < NW ? k + u : k + u + 1);
                        __builtin_amdgcn_sched_barrier(0);
                        split_multiply<FULL, MW, NW>(acc, accs, aq[u], bq[(u * NW + i) & 1], i);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    fetch_w(aq[u], k + u + PF);
                }
            }
#pragma unroll
            for (int u = 0; u < PF - 1; ++u) {
                if (main_steps + u < n) {
#pragma unroll
                    for (int i = 0; i < NW; ++i) {
                        fetch_x(bq[(u * NW + i + 1) & 1], i + 1 < NW ? i + 1 : 0, i + 1 < NW ? main_steps + u : main_steps + u + 1);
                        split_multiply<FULL, MW, NW>(acc, accs, aq[u], bq[(u * NW + i) & 1], i);
                    }
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
    split_store<true, MW * NW>([&](int t) { return acc[t % MW][t / MW]; }, [](int t, int& m, int& i) { m = t % MW; i = t / MW; return true; },
                               x, y, a, tab, b0, p0, mblk0, kg, ch_lo * a.CC, ch_hi * a.CC, position);
}

// ------------------------------------------------------------------------------------------------
// The pipelined form (producers = 4): the chunks are staged by four waves of their own into two LDS
// buffers, one chunk ahead of the eight multiplying waves, whose weights in flight never drain --
// the one-shot form above spends as long between two multiplications (refilling the weights, waiting
// for its staging, splitting) as in them on deep layers: 10 of 16.5 thousand clocks per chunk of the 1x1
// 2048-512 layer on 7 x 7 planes.  Protocol of the DENSE variant's pipelined kernel: barrier k says "chunk
// k is staged" and "chunk k - 1 has been multiplied"; it waits for LDS traffic only, so that weight loads
// stay in flight across it.  Twelve waves leave 168 registers a wave: wave tiles of at most 8 blocks.
// The steps of a wave are tabulated 64 at a time, one per lane, in both forms: worked out one after the other by the scalar unit they cost
// 10 - 15 % (us per pass of the same shape: 3x3 stride 2 512-512 at 14 x 14, batch 32 49.7 -> 43.4, 3x3 128-128 at 28 x 28 38.0 -> 35.2,
// 1-D 300-64 along 64, batch 128 10.8 -> 9.5, 3x3 100-90 at 27 x 31, batch 7 15.5 -> 14.2, 1x1 2048-512 at 7 x 7 28.0 -> 27.4).
// Two or four groups of the multiplying waves split the contraction: four where a tile is small, so that its waves do not all read the
// same weights or the same tile operands (3x3 64-64 at 32 x 32, one image: 5.4 us with two groups, 4.8 with four; eight groups were
// level there and slower elsewhere).
// ------------------------------------------------------------------------------------------------
template <int MW, int NW, int KG, int EPV, bool FULL>
__global__ void __launch_bounds__(768)
split_pipe_kernel(const float* __restrict__ x, float* __restrict__ y, const unsigned char* __restrict__ wfrag, const SplitArgs args, const SplitTable tab)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    constexpr int NTC = 512, NTP = 256;                      // multiplying, staging threads
    constexpr int PF = 2;                                    // steps of weights in flight
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave12 = __builtin_amdgcn_readfirstlane(tid >> 6);

    const SplitArgs a = args_at_once(args);
    const SplitBlock block = split_block(a);
    const int bt = block.bt, db = block.db;
    const int bg = __builtin_amdgcn_readfirstlane(sdiv(bt, a.inv_tiles_p));
    const int tpi = bt - bg * a.tiles_p;
    const int b0 = bg * a.NS, p0 = tpi * a.TP;
    const int row0 = p0 * a.s_h - a.pad_h;
    const int buf = 3 * a.bufsz;
    SplitStage st = split_stage<EPV>(a, x, b0, row0, 0);

    if (wave12 >= 8) {
        // ------------------------------------------------------------------ staging waves
        const int ptid = tid - NTC;
        constexpr int VB = kSplitVB<EPV>, per_round = NTP * VB;
        float pre[2][32];
        SplitSlot slots[2][VB];
        // two rounds of a chunk are loaded a chunk ahead, the others in place
        // (nblocks = 0: a tile that lies in the padding altogether)
        const bool one = st.nblocks > 0, two = st.nblocks > per_round;
        split_slots<EPV>(slots[0], st, a, ptid, NTP);
        if (one) split_load<EPV>(pre[0], st, slots[0]);
        split_slots<EPV>(slots[1], st, a, ptid + per_round, NTP);
        if (two) split_load<EPV>(pre[1], st, slots[1]);
        for (int k = 0; k < a.nchunks; ++k) {
            unsigned char* to = lds + (k & 1) * buf;
            if (one) split_put<EPV>(pre[0], st, to, slots[0], a);
            if (two) split_put<EPV>(pre[1], st, to, slots[1], a);
            for (int v0 = ptid + 2 * per_round; v0 - ptid < st.nblocks; v0 += per_round) {
                SplitSlot t[VB];
                split_slots<EPV>(t, st, a, v0, NTP);
                split_load<EPV>(pre[0], st, t);
                split_put<EPV>(pre[0], st, to, t, a);
            }
            if (k + 1 < a.nchunks) {
                split_advance(st, a);
                if (one) split_load<EPV>(pre[0], st, slots[0]);
                if (two) split_load<EPV>(pre[1], st, slots[1]);
            }
            split_barrier();                                 // barrier k
        }
        return;
    }

    constexpr int W1 = 8 / KG;                               // waves of one group
    const int kgrp = wave12 / W1, wave = wave12 % W1;
    const int lwm = a.bits >> 4 & 3, wm = wave & ((1 << lwm) - 1), wn = wave >> lwm;
    const int n16 = lane & 15, kg = lane >> 4;
    const int mblk0 = db * (a.DB >> 4) + wm * MW;
    const int wrow = a.RS * a.NCB * 3072;
    const unsigned char* wbase = wfrag + (int64_t)mblk0 * wrow + lane * 16;

    // The groups take steps kgrp, kgrp + KG, ... of the whole contraction (chunk, filter tap, channel block of the chunk).  64 of a
    // wave's steps are tabulated at a time, one per lane: LDS offset of the tile operands, offset of the weights, chunk.
    const int total = a.RS * a.NCB, nsteps = (total - kgrp + KG - 1) / KG;
    const int cbf = a.CC >> 5, spc = a.RS * cbf;
    const float inv_spc = __builtin_amdgcn_rcpf((float)spc), inv_cbf = __builtin_amdgcn_rcpf((float)cbf);
    const float inv_last = __builtin_amdgcn_rcpf((float)a.cbs_last), inv_S = __builtin_amdgcn_rcpf((float)a.S);
    int xtab, wtab, ctab, nbar = 0;
    auto table = [&](int s0) __attribute__((always_inline)) {
        const int s = min(kgrp + KG * (s0 + lane), total - 1);
        ctab = sdiv(s, inv_spc);
        const bool lastc = ctab == a.nchunks - 1;
        const int rem = s - ctab * spc, tap = sdiv(rem, lastc ? inv_last : inv_cbf), cb = rem - tap * (lastc ? a.cbs_last : cbf);
        const int r = sdiv(tap, inv_S);
        xtab = (ctab & 1) * buf + (r * a.Ws + tap - r * a.S) * a.pitch + cb * 64;
        wtab = tap * a.NCB + ctab * cbf + cb;
    };
    uint4w aq[PF][MW][3], bq[2][3];
    auto fetch_w = [&](uint4w (&av)[MW][3], int k) __attribute__((always_inline)) {
        const unsigned char* wu = wbase + (int64_t)__builtin_amdgcn_readlane(wtab, min(k, 63)) * 3072;
#pragma unroll
        for (int m = 0; m < MW; ++m)
#pragma unroll
            for (int t = 0; t < 3; ++t) av[m][t] = *reinterpret_cast<const uint4w*>(wu + m * wrow + t * 1024);
    };
    table(0);
#pragma unroll
    for (int u = 0; u < PF; ++u) fetch_w(aq[u], u);
    // the padding of both buffers is written once, behind the first weight requests
    __builtin_amdgcn_sched_barrier(0);
    split_pad(lds, tid, NTC, st, a);
    if (a.nchunks > 1) split_pad(lds + buf, tid, NTC, st, a);

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
    for (int s0 = 0; s0 < nsteps; s0 += 64) {
        const int n = min(64, nsteps - s0);
        if (s0 > 0) {
            table(s0);
#pragma unroll
            for (int u = 0; u < PF; ++u) fetch_w(aq[u], u);
        }
        auto fetch_x = [&](uint4w (&bv)[3], int i, int k) __attribute__((always_inline)) {
            k = min(k, n - 1);
            if (i == 0) {
                const int ch = __builtin_amdgcn_readlane(ctab, k);
                while (nbar <= ch) { split_barrier(); ++nbar; }      // the chunk of this step is staged
            }
            const int off = bbase[i] + __builtin_amdgcn_readlane(xtab, k);
#pragma unroll
            for (int t = 0; t < 3; ++t) bv[t] = *reinterpret_cast<const uint4w*>(lds + off + t * a.bufsz);
        };
        fetch_x(bq[0], 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        const int main_steps = n / PF * PF;
        for (int k = 0; k < main_steps; k += PF) {
#pragma unroll
            for (int u = 0; u < PF; ++u) {
#pragma unroll
                for (int i = 0; i < NW; ++i) {
                    fetch_x(bq[(u * NW + i + 1) & 1], i + 1 < NW ? i + 1 : 0, i + 1 < NW ? k + u : k + u + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    split_multiply<FULL, MW, NW>(acc, accs, aq[u], bq[(u * NW + i) & 1], i);
                    __builtin_amdgcn_sched_barrier(0);
                }
                fetch_w(aq[u], k + u + PF);
            }
        }
        if (main_steps < n) {
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                if (i + 1 < NW) fetch_x(bq[(i + 1) & 1], i + 1, main_steps);
                split_multiply<FULL, MW, NW>(acc, accs, aq[0], bq[i & 1], i);
            }
        }
    }
    while (nbar < a.nchunks) { split_barrier(); ++nbar; }    // (a wave without steps in the last chunks)
#pragma unroll
    for (int m = 0; m < MW; ++m)
#pragma unroll
        for (int i = 0; i < NW; ++i) acc[m][i] += accs[m][i];
    // The groups meet in LDS (the staging waves have ended): block b is added up and stored by group b mod KG, the others give it
    // theirs, a lane's own 16 bytes per block.
    __syncthreads();
    constexpr int NB = MW * NW, BPW = (NB + KG - 1) / KG;
    float4v* ex = reinterpret_cast<float4v*>(lds) + wave * (NB * (KG - 1) * 64) + lane;
#pragma unroll
    for (int b = 0; b < NB; ++b)
        if (kgrp != b % KG) ex[(b * (KG - 1) + ((kgrp - b % KG - 1) & (KG - 1))) * 64] = acc[b % MW][b / MW];
    __syncthreads();
    float4v sum[BPW];
    auto owned = [&](int t, int& m, int& i) {
        const int b = kgrp + t * KG;
        m = b % MW;
        i = b / MW;
        return b < NB;
    };
#pragma unroll
    for (int t = 0; t < BPW; ++t) {
#pragma unroll
        for (int g = 0; g < KG; ++g)
            if (g == 0 || (t * KG + g < NB && kgrp == g)) sum[t] = acc[(t * KG + g) % MW][(t * KG + g) / MW];
        if (kgrp + t * KG < NB) {
#pragma unroll
            for (int q = 0; q < KG - 1; ++q) sum[t] += ex[((kgrp + t * KG) * (KG - 1) + q) * 64];
        }
    }
    split_store<false, BPW>([&](int t) { return sum[t]; }, owned, x, y, a, tab, b0, p0, mblk0, kg, 0, a.C, position);
}

template <int MW, int NW, int KG, int EPV, bool FULL>
static sc_status_t launch_split_full(const Plan& p, const SplitArgs& a, const SplitTable& tab, const void* x, void* y, int grid, hipStream_t stream)
{
    // KG > 2: the pipelined form (eight multiplying waves and four that stage), KG - 10 groups
    auto kernel = [] {
        if constexpr (KG > 2) return &split_pipe_kernel<MW, NW, KG - 10, EPV, FULL>;
        else return &split_conv_kernel<MW, NW, KG, EPV, FULL>;
    }();
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [&] {
        attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes);
    });
    if (attr_err != hipSuccess) return SC_ERR_HIP;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(KG > 2 ? 768 : 256 * KG), p.mg.lds_bytes, stream, static_cast<const float*>(x),
                       static_cast<float*>(y), p.d_wfrag, a, tab);
    return hipGetLastError() == hipSuccess ? SC_OK : SC_ERR_HIP;
}

template <int KG, int EPV, int MW, int NW>
static sc_status_t launch_split_one(const Plan& p, const SplitArgs& a, const SplitTable& t, const void* x, void* y, int grid, hipStream_t stream)
{
    return p.split_full ? launch_split_full<MW, NW, KG, EPV, true>(p, a, t, x, y, grid, stream)
                        : launch_split_full<MW, NW, KG, EPV, false>(p, a, t, x, y, grid, stream);
}

template <int KG, int EPV>
static sc_status_t launch_split_typed(const Plan& p, const SplitArgs& a, const SplitTable& t, const void* x, void* y, int grid, hipStream_t stream)
{
    switch (p.mg.MW * 10 + p.mg.NW) {
        case 11: return launch_split_one<KG, EPV, 1, 1>(p, a, t, x, y, grid, stream);
        case 12: return launch_split_one<KG, EPV, 1, 2>(p, a, t, x, y, grid, stream);
        case 14: return launch_split_one<KG, EPV, 1, 4>(p, a, t, x, y, grid, stream);
        case 17: return launch_split_one<KG, EPV, 1, 7>(p, a, t, x, y, grid, stream);
        case 18: return launch_split_one<KG, EPV, 1, 8>(p, a, t, x, y, grid, stream);
        case 21: return launch_split_one<KG, EPV, 2, 1>(p, a, t, x, y, grid, stream);
        case 22: return launch_split_one<KG, EPV, 2, 2>(p, a, t, x, y, grid, stream);
        case 24: return launch_split_one<KG, EPV, 2, 4>(p, a, t, x, y, grid, stream);
        case 27: if constexpr (KG <= 2) return launch_split_one<KG, EPV, 2, 7>(p, a, t, x, y, grid, stream); break;
    }
    return SC_ERR_UNSUPPORTED;
}

}  // namespace sc
