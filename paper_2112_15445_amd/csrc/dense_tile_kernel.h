// The one-shot kernel of the DENSE variant: the tile is staged transposed, a chunk of input channels at a
// time, by all waves, and multiplied by all of them.  See dense_mfma.hip for the formulation.
//
// What bounds the layers that it serves is not the matrix pipe (22 clocks per 16 x 16 x 32 instruction) but what
// happens around it, so the kernel is laid out for short phases:
//   * the loads of the first chunk are requested before anything else is worked out; weights, LDS zeroing, the
//     lanes' positions and the table of steps are prepared while they are on their way;
//   * staging moves whole registers: blocks of 8 (16) channels x up to 8 columns, transposed by byte
//     permutations; of 16 neighbouring lanes, four take neighbouring blocks of one channel group and the next fours the next
//     channel groups.  The address unit joins only neighbouring lanes to lines, so that a load wants as many of them
//     along a row as it can get, while the 16-byte LDS writes of 16 lanes want different 16-byte banks: with four
//     channel groups beside each other they have them for blocks of 4 columns, and pairs share one for 8 and 2 columns and
//     mostly for 1 (all 16 lanes along a row of 8-column blocks would share two; four channel groups on every four lanes, the
//     first arrangement here, read a quarter of a line for each lane group);
//   * weights come through the vector L1, which gives a CU 39 bytes a clock with four waves and 45 with eight, from four
//     loads in flight on and whatever the region (loads of 1 KB a wave alone, regions of 16 KB to 4 MB: 82 and 94 - 98 GB/s a
//     CU at 2.1 GHz): what a workgroup reads of them is what counts.  The eight waves may therefore
//     split the contraction up to eight ways (KG) over one tile of outputs instead of fetching the
//     same weights for several tiles; their sums meet in LDS;
//   * the operands are exchanged (positions are the rows of the matrix instruction, channels its columns), so
//     that a lane holds four neighbouring positions of one channel and stores them as one word.
//   * a step costs a wave little but its matrix instructions: its LDS offset and its place in the weights come from lanes of two registers, and
//     the weights are read at 32-bit offsets from scalar bases (12 scalar instructions less a step: the int8 layers below 109.3 -> 106.1 us
//     of the same shapes, 4b/16b 512-512 11.1 -> 10.9, f16 64-64 15.1 -> 14.8);
//   * a launch reads its arguments at once (TileArgs), staging is instantiated by the columns of a load, and the first chunk is staged
//     ahead of the loop over the chunks, so that the compiler knows how many loads are in flight and waits for the input only, not for the weights behind it.
// Measured per pass, before and after the last of these: f16 3x3 64-64 at 56 x 56, batch 32 14.9, 14.5 us; f16 3x3 256-256 at 14 x 14,
// batch 32 13.6, 13.0; 4b/16b 3x3 512-512 at 4 x 4, batch 64 11.9, 10.9; the 13 int8 layers of VGG-16, batch 64 121, 111 (a layer launched alone again and
// again 9.3, 7.5 in the mean: in the stack about 1.5 us of each launch are the first pass through its code).  More weights in flight (8 and 12 steps) are
// slower: they compete with the input when a workgroup starts (112 us for the int8 layers).
#pragma once

#include "dense_mfma_kernel.h"

namespace sc {

// ------------------------------------------------------------------------------------------------
// Staging.  One block = CV channels x EPV columns of one run (an input row; or, where the staged rows carry no
// padding columns, all of them).  A run that is no multiple of EPV ends in a block that starts EPV before its end: the
// columns that two blocks share are written twice with the same values.  The loads therefore have any
// alignment that an element has.  A round is one load of 32 registers per thread.
// ------------------------------------------------------------------------------------------------
struct TileStage {
    const char* xs;              // first staged element of sample 0, channel 0 of the chunk
    unsigned sample_b, plane_b, row_b;   // bytes per sample, channel and input row
    int nblocks, rowsG, per_cg, quads, G, run, cleft, dst0;      // blocks (dead ones of the last quad of a channel group too)
    int npos1, Ws;
    bool whole;                  // every channel of the chunk's groups exists in the layer
    float inv_quads, inv_rowsG, inv_G;
};

__device__ __forceinline__ int tdiv(int e, float inv) { return (int)__builtin_fmaf((float)e, inv, 0.5f * inv); }   // as fdiv19

template <typename X> constexpr int kTileCV = 16 / (int)sizeof(X);
template <typename X, int EPV> constexpr int kTileWPE = EPV * (int)sizeof(X) >= 4 ? EPV * (int)sizeof(X) / 4 : 1;
template <typename X, int EPV> constexpr int kTileVB = 32 / (kTileCV<X> * kTileWPE<X, EPV>);    // blocks per thread and round

// Where a block is read from (bytes from st.xs in the first channel group's first channel, and its channel) and written to
// (bytes into the LDS image; -1: no such block, then the first block of the first channel groups is read).  The same for
// every chunk.
struct TileSlot { unsigned off; int cg, dst; };

template <typename X, int EPV>
__device__ __forceinline__ TileSlot tile_slot(const TileStage& st, int pitch, int v)
{
    int cg4 = tdiv(v >> 4, st.inv_quads);
    int r = ((v >> 4) - cg4 * st.quads) * 4 + (v & 3);
    const bool live = v < st.nblocks && r < st.per_cg;
    if (!live) cg4 = r = 0;
    const int cg = cg4 * 4 + (v >> 2 & 3);
    int sm = 0, ii = 0;
    if (st.rowsG != st.per_cg) { sm = tdiv(r, st.inv_rowsG); r -= sm * st.rowsG; }
    if (st.rowsG != st.G) { ii = tdiv(r, st.inv_G); r -= ii * st.G; }
    const int col = min(r * EPV, st.run - EPV);
    return {(unsigned)sm * st.sample_b + (unsigned)ii * st.row_b + (unsigned)col * (unsigned)sizeof(X), cg,
            live ? (sm * st.npos1 + st.dst0 + ii * st.Ws + col) * pitch + cg * 16 : -1};
}

// Address of a staging load, whole in the lane's registers.  Left to itself the compiler takes the scalar base and the 32-bit
// offset apart (global_load v, v, s[]), and loads in that form that are not aligned to their width are slower than
// those from a 64-bit lane address, 16.4 us for 13.6 (4-bit 1x1 1633-18 at 15 x 14, batch 58, rows of 210 bytes),
// 10.7 for 9.2 (f16 3x3 33-93 at 13 x 13, batch 20, tuned for two rows a tile); aligned ones are level.
using TileSrc = const __attribute__((address_space(1))) char*;
__device__ __forceinline__ TileSrc tile_src(const char* base, unsigned off)
{
    uint64_t ad = reinterpret_cast<uint64_t>(base) + off;
    asm("" : "+v"(ad));
    return reinterpret_cast<TileSrc>(ad);
}

template <typename X, int EPV>
__device__ __forceinline__ void tile_load(unsigned (&pre)[32], const TileStage& st, const TileSlot (&slot)[kTileVB<X, EPV>])
{
    constexpr int CV = kTileCV<X>, W = kTileWPE<X, EPV>, VB = kTileVB<X, EPV>, B = EPV * (int)sizeof(X);
#pragma unroll
    for (int u = 0; u < VB; ++u) {
        unsigned off = slot[u].off;
        int cg = slot[u].cg;
        // (opaque: the addresses of a block are worked out again for every chunk, not kept in registers)
        asm volatile("" : "+v"(off), "+v"(cg));
        // (of any alignment: one load each all the same)
        auto load = [&](int j, TileSrc src) __attribute__((always_inline)) {
            if constexpr (B >= 4) {
                unsigned e[W];
                __builtin_memcpy(e, (const void*)src, B);
#pragma unroll
                for (int w = 0; w < W; ++w) pre[(u * CV + j) * W + w] = e[w];
            } else if constexpr (B == 2) {
                unsigned short e;
                __builtin_memcpy(&e, (const void*)src, 2);
                pre[u * CV + j] = e;
            } else {
                pre[u * CV + j] = *reinterpret_cast<const __attribute__((address_space(1))) unsigned char*>(src);
            }
        };
        if (st.whole) {
            // (one 64-bit addition from channel to channel)
            TileSrc src = tile_src(st.xs, off + (unsigned)(cg * CV) * st.plane_b);
#pragma unroll
            for (int j = 0; j < CV; ++j) {
                load(j, src);
                src += st.plane_b;
                asm("" : "+v"(src));
                __builtin_amdgcn_sched_barrier(0);           // (one address at a time: registers)
            }
        } else {
            unsigned o = off + (unsigned)(cg * CV) * st.plane_b;
#pragma unroll
            for (int j = 0; j < CV; ++j) {
                // (channels past the layer's last: the block's place in channel 0, zeroed when it is stored)
                load(j, tile_src(st.xs, cg * CV + j < st.cleft ? o : off));
                o += st.plane_b;
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
}

template <typename X, int EPV>
__device__ __forceinline__ void tile_store(unsigned (&pre)[32], const TileStage& st, unsigned char* lds, int pitch, const TileSlot (&slot)[kTileVB<X, EPV>])
{
    constexpr int CV = kTileCV<X>, W = kTileWPE<X, EPV>, VB = kTileVB<X, EPV>;
    constexpr int EPW = 4 / (int)sizeof(X);                  // columns per register
#pragma unroll
    for (int u = 0; u < VB; ++u) {
        if (slot[u].dst < 0) continue;
        int cg = slot[u].cg, to = slot[u].dst;
        asm volatile("" : "+v"(cg), "+v"(to));
        unsigned char* dst = lds + to;
        if (!st.whole) {
#pragma unroll
            for (int j = 0; j < CV; ++j)
                if (cg * CV + j >= st.cleft) {
#pragma unroll
                    for (int w = 0; w < W; ++w) pre[(u * CV + j) * W + w] = 0u;
                }
        }
#pragma unroll
        for (int w = 0; w < W; ++w) {
            if constexpr (sizeof(X) == 2) {
#pragma unroll
                for (int e = 0; e < (EPV < EPW ? EPV : EPW); ++e) {
                    uint4w o;
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        o[q] = __builtin_amdgcn_perm(pre[(u * CV + 2 * q + 1) * W + w], pre[(u * CV + 2 * q) * W + w], e ? 0x07060302u : 0x05040100u);
                    *reinterpret_cast<uint4w*>(dst + (w * EPW + e) * pitch) = o;
                }
            } else {
                // 4 x 4 bytes of 4 channels at a time: pairs of channels first, then pairs of pairs
                uint4w o[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const unsigned c0 = pre[(u * CV + 4 * q) * W + w], c1 = pre[(u * CV + 4 * q + 1) * W + w];
                    const unsigned c2 = pre[(u * CV + 4 * q + 2) * W + w], c3 = pre[(u * CV + 4 * q + 3) * W + w];
                    const unsigned a0 = __builtin_amdgcn_perm(c1, c0, 0x05010400u), b0 = __builtin_amdgcn_perm(c3, c2, 0x05010400u);
                    o[0][q] = __builtin_amdgcn_perm(b0, a0, 0x05040100u);
                    o[1][q] = __builtin_amdgcn_perm(b0, a0, 0x07060302u);
                    if constexpr (EPV >= 4) {
                        const unsigned a1 = __builtin_amdgcn_perm(c1, c0, 0x07030602u), b1 = __builtin_amdgcn_perm(c3, c2, 0x07030602u);
                        o[2][q] = __builtin_amdgcn_perm(b1, a1, 0x05040100u);
                        o[3][q] = __builtin_amdgcn_perm(b1, a1, 0x07060302u);
                    }
                }
#pragma unroll
                for (int e = 0; e < (EPV < 4 ? EPV : 4); ++e) *reinterpret_cast<uint4w*>(dst + (w * 4 + e) * pitch) = o[e];
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------
// Stores of four neighbouring positions of one output channel (of any alignment that an element has).  Not with the
// non-temporal hint: a wave's store covers 32 bytes (f16) of each of 16 channels, and the hint keeps L2 from joining
// the neighbouring blocks to whole lines (f16 1x1 128-512 at 28 x 28, batch 32: 28.4 us with it, 18.8 without).
// ------------------------------------------------------------------------------------------------
template <typename A> __device__ __forceinline__ A tile_max(A p, A q)
{
    if constexpr (std::is_same<A, float>::value) return __builtin_fmaxf(p, q);
    else return p > q ? p : q;
}

__device__ __forceinline__ int8_t tile_code(int v, float rq)
{
    const float q = rintf(__int2float_rn(v) * rq);
    return (int8_t)(int)fminf(fmaxf(q, -127.0f), 127.0f);
}

template <sc_dtype_t DT, typename Acc>
__device__ __forceinline__ void tile_put4(typename Types<DT>::Y* __restrict__ y, int64_t off, Acc v, bool relu, bool codes, float rq, int count)
{
    if (relu) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const typename Types<DT>::A e = v[j];
            v[j] = tile_max(e, typename Types<DT>::A(0));
        }
    }
    if constexpr (kIntActs<DT>) {
        if (codes) {
            int8_t* yc = reinterpret_cast<int8_t*>(y) + off;
            if (count >= 4) {
                const unsigned w = (unsigned)(uint8_t)tile_code(v[0], rq) | (unsigned)(uint8_t)tile_code(v[1], rq) << 8 |
                                   (unsigned)(uint8_t)tile_code(v[2], rq) << 16 | (unsigned)(uint8_t)tile_code(v[3], rq) << 24;
                typedef unsigned __attribute__((aligned(1))) U;
                *reinterpret_cast<U*>(yc) = w;
            } else {
#pragma unroll
                for (int j = 0; j < 3; ++j)
                    if (j < count) yc[j] = tile_code(v[j], rq);
            }
            return;
        }
        if (count >= 4) {
            typedef int4v_ __attribute__((aligned(4))) U;
            *reinterpret_cast<U*>(y + off) = v;
        } else {
#pragma unroll
            for (int j = 0; j < 3; ++j)
                if (j < count) store_out(y + off + j, v[j]);
        }
    } else {
        if (count >= 4) {
            typedef unsigned V2 __attribute__((ext_vector_type(2)));
            typedef V2 __attribute__((aligned(2))) U;
            V2 w;
#pragma unroll
            for (int j = 0; j < 2; ++j)
                w[j] = (unsigned)__half_as_ushort(narrow<DT>(v[2 * j])) | (unsigned)__half_as_ushort(narrow<DT>(v[2 * j + 1])) << 16;
            *reinterpret_cast<U*>(y + off) = w;
        } else {
#pragma unroll
            for (int j = 0; j < 3; ++j)
                if (j < count) store_out(y + off + j, narrow<DT>(v[j]));
        }
    }
}

// Workgroup -> (tile of positions bt, block of output channels db of ndb).  Workgroups are dealt round-robin to
// the 8 XCDs: they are renumbered so that each XCD gets a contiguous run.  Within it either the blocks of one tile
// are neighbours (they find the tile in the L2 that their siblings loaded), or, where the weights outweigh the
// input (bit 0), the tiles of one block: an XCD then streams its share of the weights and not all of them.
// Both indices are chosen by value and made wave-uniform: written through references in two branches they went
// through scratch memory, a store and a load before the first address could be formed, and everything derived from them
// was vector arithmetic (all 26 tile kernels: 12 bytes of scratch and 15 - 18 vector registers more).
struct TileBlock { int bt, db; };
__device__ __forceinline__ TileBlock tile_block(const TileArgs& a)
{
    const int xcd = blockIdx.x & 7;
    const int wg = xcd * a.gq + min(xcd, a.gr) + (int)(blockIdx.x >> 3);
    const int hi = __builtin_amdgcn_readfirstlane(fdiv19(wg, a.inv_inner)), lo = wg - hi * a.inner;
    return {a.bits & 1 ? lo : hi, a.bits & 1 ? hi : lo};
}

// WIDE: a 16-row block of the weights is 4 GB or more (filter taps x channel blocks of 2^22 and more: 134 million input channels x taps in 16 bits),
// and its steps are addressed in 64 bits.  Instantiated for one column a load only.
template <sc_dtype_t DT, int MW, int NW, int LEPV, bool WIDE>
__global__ void __launch_bounds__(512, 2)
mfma_tile_kernel(const typename Types<DT>::X* __restrict__ x, typename Types<DT>::Y* __restrict__ y,
                 const uint4w* __restrict__ wfrag, const TileArgs args)
{
    using X = typename Types<DT>::X;
    using A = typename Types<DT>::A;
    using Acc = typename std::conditional<kIntActs<DT>, int4v_, float4v>::type;
    constexpr int CB = kChanBlock<DT>, CV = kChanVec<DT>;
    constexpr int PF = MW >= 2 ? 4 : 8;                      // steps of weights in flight
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];

    const TileArgs a = args_at_once(args);
    constexpr int lepv = LEPV;                               // log2 of the columns per staging load
    const int lwm = a.bits >> 6 & 3, lwn = a.bits >> 8 & 3, lkg = a.bits >> 10 & 3;
    const int NT = (a.bits >> 12 & 15) * 64;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, kg = lane >> 4;

    const TileBlock block = tile_block(a);
    const int bt = block.bt, db = block.db;
    const int bg = __builtin_amdgcn_readfirstlane(fdiv19(bt, a.inv_tiles_p));
    const int tpi = bt - bg * a.tiles_p;
    const int b0 = bg * a.NS, p0 = tpi * a.TP;
    const int row0 = p0 * a.s_h - a.pad_h;

    // ---------------------------------------------------------------- the loads of the first chunk
    TileStage st;
    const int nsv = min(a.NS, a.N - b0);                     // samples inside the batch
    const int ilo = max(0, -row0);                           // staged rows inside the input: [ilo, ilo + nrows)
    const int nrows = max(0, min(a.Hs, a.H - row0) - ilo);
    {
        const bool flat = a.bits & 2;
        const int rows = flat ? min(nrows, 1) : nrows;
        st.run = flat ? nrows * a.W : a.wcols;
        st.G = (st.run + (1 << lepv) - 1) >> lepv;
        st.rowsG = rows * st.G;
        st.per_cg = nsv * st.rowsG;
        st.quads = (st.per_cg + 3) >> 2;
        st.nblocks = (int)((unsigned)a.CC / CV) * st.quads * 4;
        st.inv_quads = __builtin_amdgcn_rcpf((float)max(st.quads, 1));
        st.inv_rowsG = __builtin_amdgcn_rcpf((float)max(st.rowsG, 1));
        st.inv_G = __builtin_amdgcn_rcpf((float)max(st.G, 1));
        st.dst0 = ilo * a.Ws + a.pad_w;
        st.npos1 = a.npos1;
        st.Ws = a.Ws;
        st.plane_b = a.plane_b;
        st.sample_b = a.sample_b;
        st.row_b = (unsigned)a.W * (unsigned)sizeof(X);
        st.xs = reinterpret_cast<const char*>(x) + (int64_t)b0 * st.sample_b + (int64_t)(row0 + ilo) * st.row_b;
        st.cleft = a.C;
        st.whole = st.cleft >= a.CC;
    }
    // One round of a chunk is loaded a chunk ahead.  (Two, the form before, cost 32 registers and half of the code -- 80 KB for the
    // largest wave tiles, where 14 and 16 blocks now take 38 - 49 in 16 and 56 - 65 in 8 bits, of the 64 KB of the instruction cache of two
    // CUs: f16 3x3 64-64 at 56 x 56, batch 32 15.4 -> 15.0 us, the 13 int8 layers of VGG-16, batch 64 110.9 -> 108.3, other layers level.
    // 108 - 139 registers for the wave tiles of up to four blocks, but 4 x 1 blocks with 153 - 174, leave room for three or four waves per
    // SIMD, which layers with many short workgroups need to overlap them: 4b/16b 3x3 80-383 at 6 x 6, batch 128, 15.8 us with two waves,
    // 12.4 with three.  1 x 7, 1 x 8 and 2 x 4 blocks with 138 - 157 leave it for three.)
    constexpr int EPV = 1 << LEPV, VB = kTileVB<X, EPV>;
    unsigned pre[32];
    TileSlot slots[VB];
    const int per_round = NT * VB;
    auto locate = [&](TileSlot (&t)[VB], int v0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < VB; ++u) t[u] = tile_slot<X, EPV>(st, a.pitch, v0 + u * NT);
    };
    // (nblocks = 0: a tile that lies in the padding altogether)
    if (st.nblocks) {
        locate(slots, tid);
        tile_load<X, EPV>(pre, st, slots);
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---------------------------------------------------------------- roles of the waves
    const int wm = wave & ((1 << lwm) - 1), wn = (wave >> lwm) & ((1 << lwn) - 1), kgrp = wave >> (lwm + lwn);
    const int KG = 1 << lkg;
    const int mblk0 = db * (a.DB >> 4) + wm * MW;
    // requantisation multipliers of this lane's channels (n16 of each row block), requested with the input: read where they are
    // used they cost a pooled layer a trip to memory for every channel that a thread finishes
    float rqs[MW];
#pragma unroll
    for (int m = 0; m < MW; ++m) rqs[m] = 0.0f;
    if constexpr (kIntActs<DT>) {
        // (through a global pointer: a load that might be from LDS would have to be waited for with everything else)
        const auto* from = (const __attribute__((address_space(1))) float*)a.requant;
#pragma unroll
        for (int m = 0; m < MW; ++m) rqs[m] = from[min((mblk0 + m) * 16 + n16, a.D - 1)];
    }
    const int64_t wrow = (int64_t)(a.RS * a.NCB) << 10;      // bytes per 16-row block of the weights
    const unsigned char* wrows = reinterpret_cast<const unsigned char*>(wfrag) + mblk0 * wrow;

    // Steps of a chunk: filter tap, then channel block of the chunk; this wave takes kgrp, kgrp + KG, ...
    // Up to 56 of them are tabulated one per lane (LDS offset of the tile operands, bytes into a row block of the weights) and
    // read back with v_readlane; the lanes past the last repeat it: operands are requested up to 8 steps ahead, without a test.
    int xtab;
    unsigned wtab;
    constexpr int kTable = 56;                               // (a multiple of PF, and 8 lanes more)
    auto table = [&](int s0, int n, int cbs, int gcb0) {
        const int s = min(kgrp + KG * (s0 + min(lane, max(n, 1) - 1)), a.RS * cbs - 1);
        const int tap = tdiv(s, cbs == (int)((unsigned)a.CC / CB) ? a.inv_ccb : a.inv_cbs_last);
        const int cb = s - tap * cbs;
        const int r = tdiv(tap, a.inv_S);
        const int sx = tap - r * a.S;
        xtab = (r * a.Ws + sx) * a.pitch + cb * 64;
        wtab = (unsigned)(tap * a.NCB + gcb0 + cb) << (WIDE ? 0 : 10);
    };
    uint4w aq[PF][MW], bq[4];
    auto fetch_w = [&](uint4w (&av)[MW], int s) __attribute__((always_inline)) {
        if constexpr (WIDE) {
            const unsigned char* ws = wrows + ((uint64_t)(unsigned)__builtin_amdgcn_readlane((int)wtab, s) << 10);
#pragma unroll
            for (int m = 0; m < MW; ++m) av[m] = *reinterpret_cast<const uint4w*>(ws + m * wrow + (unsigned)lane * 16u);
        } else {
            // (32-bit offsets from a scalar base for each row block)
            const unsigned off = (unsigned)__builtin_amdgcn_readlane((int)wtab, s) + (unsigned)lane * 16u;
#pragma unroll
            for (int m = 0; m < MW; ++m) av[m] = *reinterpret_cast<const uint4w*>(wrows + m * wrow + off);
        }
    };
    // steps of this wave in a chunk of cbs channel blocks
    auto steps_of = [&](int cbs) { const int all = a.RS * cbs; return all > kgrp ? (all - kgrp + KG - 1) >> lkg : 0; };
    auto start_w = [&](int s0, int n, int cbs, int gcb0) __attribute__((always_inline)) {
        table(s0, min(kTable, n - s0), cbs, gcb0);
#pragma unroll
        for (int u = 0; u < PF; ++u) fetch_w(aq[u], u);
    };
    int cbs = min(a.CC, a.NCB * CB) / CB;
    int nsteps = steps_of(cbs);
    // (A wave without steps requests weights all the same, here and below: behind loads that only some waves issue
    // the compiler no longer knows how many are in flight, and waits for the weights before it stages the input.)
    start_w(0, nsteps, cbs, 0);
    __builtin_amdgcn_sched_barrier(0);

    // ---------------------------------------------------------------- padding: zeros, once for all chunks.  Only the positions that the
    // input does not reach, so that it and the staging need not wait for each other: threads lie as (group of 16-byte words, position).
    // (Clearing the whole image took a 512-thread workgroup 1.5 us of its first 3 at 75 KB.)
    if (a.zero) {
        const int words = (int)((unsigned)a.CC / CV), pw = a.zero >> 16, groups = NT >> pw;      // (positions, rounded up to 2^pw <= NT)
        const int first = tid >> pw;
        for (int pos = tid & ((1 << pw) - 1); pos < (a.zero & 0xffff); pos += 1 << pw) {
            const int sm = tdiv(pos, a.inv_npos1);
            const int rem = pos - sm * a.npos1;
            const int i = tdiv(rem, a.inv_Ws);
            const int w = rem - i * a.Ws;
            const bool inside = sm < nsv && (unsigned)(i - ilo) < (unsigned)nrows && (unsigned)(w - a.pad_w) < (unsigned)a.wcols;
            if (!inside)
                for (int cg = first; cg < words; cg += groups) *reinterpret_cast<uint4w*>(lds + pos * a.pitch + cg * 16) = uint4w{0u, 0u, 0u, 0u};
        }
    }

    // positions of this lane's NW column blocks in the tile image (with its k group)
    int bbase[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const int f = (wn * NW + i) * 16 + n16;
        const int sm = tdiv(f, a.inv_TPQ);
        const int rem = f - sm * a.TPQ;
        const int tp = tdiv(rem, a.inv_Q);
        const int tq = rem - tp * a.Q;
        const bool ok = f < a.npos;
        bbase[i] = (ok ? (sm * a.npos1 + tp * a.s_h * a.Ws + tq * a.s_w) * a.pitch : 0) + kg * 16;
    }
    Acc acc[MW][NW];
#pragma unroll
    for (int m = 0; m < MW; ++m)
#pragma unroll
        for (int i = 0; i < NW; ++i) acc[m][i] = Acc{0, 0, 0, 0};

    // the rest of a chunk, once its first rounds have been loaded
    auto stage = [&]() __attribute__((always_inline)) {
        if (st.nblocks) tile_store<X, EPV>(pre, st, lds, a.pitch, slots);
        for (int v0 = tid + per_round; v0 - tid < st.nblocks; v0 += per_round) {
            TileSlot t[VB];
            locate(t, v0);
            tile_load<X, EPV>(pre, st, t);
            tile_store<X, EPV>(pre, st, lds, a.pitch, t);
        }
    };
    // (the first chunk ahead of the loop, so that the compiler knows there which loads are in flight)
    stage();
    lds_barrier();
    for (int ch = 0;; ++ch) {
        if (ch + 1 < a.nchunks) {
            st.xs += (int64_t)a.CC * st.plane_b;
            st.cleft -= a.CC;
            st.whole = st.cleft >= a.CC;
            if (st.nblocks) tile_load<X, EPV>(pre, st, slots);
        }
        __builtin_amdgcn_sched_barrier(0);
        // ------------------------------------------------------------ multiply
        const int gcb0 = ch * (int)((unsigned)a.CC / CB);
        for (int s0 = 0; s0 < nsteps; s0 += kTable) {
            const int n = min(kTable, nsteps - s0);
            if (s0 > 0) start_w(s0, nsteps, cbs, gcb0);
            // operands of the tile: block b of the sequence (step, position block) goes to slot b mod 4, requested three
            // blocks ahead of its use
#pragma unroll
            for (int b = 0; b < 3; ++b)
                bq[b] = *reinterpret_cast<const uint4w*>(lds + bbase[b % NW] + __builtin_amdgcn_readlane(xtab, b / NW));
            auto step = [&](int k, int u, bool refill) __attribute__((always_inline)) {
                constexpr int AH = (NW + 2) / NW;            // steps that the requests reach ahead
                int toff[AH + 1];
#pragma unroll
                for (int q = 0; q <= AH; ++q) toff[q] = __builtin_amdgcn_readlane(xtab, k + q);
#pragma unroll
                for (int i = 0; i < NW; ++i) {
                    bq[(u * NW + i + 3) & 3] = *reinterpret_cast<const uint4w*>(lds + bbase[(i + 3) % NW] + toff[(i + 3) / NW]);
                    __builtin_amdgcn_sched_barrier(0);
                    const uint4w bv = bq[(u * NW + i) & 3];
#pragma unroll
                    for (int m = 0; m < MW; ++m) {
                        if constexpr (kIntActs<DT>)
                            acc[m][i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(int4v_, bv), __builtin_bit_cast(int4v_, aq[u][m]), acc[m][i], 0, 0, 0);
                        else
                            acc[m][i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8v, bv), __builtin_bit_cast(half8v, aq[u][m]), acc[m][i], 0, 0, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (refill) fetch_w(aq[u], k + PF);
            };
            const int main_steps = n / PF * PF;
            for (int k = 0; k < main_steps; k += PF) {
#pragma unroll
                for (int u = 0; u < PF; ++u) step(k + u, u, true);
            }
#pragma unroll
            for (int u = 0; u < PF - 1; ++u)
                if (main_steps + u < n) step(main_steps + u, u, false);
        }
        if (ch + 1 >= a.nchunks) break;
        cbs = min(a.CC, a.NCB * CB - (ch + 1) * a.CC) / CB;
        nsteps = steps_of(cbs);
        start_w(0, nsteps, cbs, gcb0 + (int)((unsigned)a.CC / CB));
        lds_barrier();                                       // the chunk has been multiplied
        stage();
        lds_barrier();
    }

    // ---------------------------------------------------------------- the outputs: a lane holds the positions 4 kg .. 4 kg + 3 of a
    // block for channel n16 of the row block
    const int PQ = a.P * a.Q;
    const int nvalid = (a.NS == 1 ? min(a.TP, a.P - p0) : a.P) * a.Q;      // positions of a sample that exist
    auto multiplier = [&](int m) __attribute__((always_inline)) {
        float rq = rqs[0];
        if constexpr (MW > 1) rq = m == 1 ? rqs[1] : rq;
        if constexpr (MW > 2) rq = m == 2 ? rqs[2] : (m == 3 ? rqs[3] : rq);
        return rq;
    };
    const bool relu = a.bits & 4, codes = a.bits & 1 << 16;
    auto put = [&](int m, int i, const Acc& v, float rq) __attribute__((always_inline)) {
        const int d = (mblk0 + m) * 16 + n16;
        const int f = (wn * NW + i) * 16 + 4 * kg;
        if (d >= a.D) return;
        if (a.NS == 1) {
            const int count = min(nvalid - f, 4);
            if (count > 0) tile_put4<DT>(y, ((int64_t)b0 * a.D + d) * PQ + p0 * a.Q + f, v, relu, codes, rq, count);
        } else {
            // whole planes of several samples: a group of four that reaches into the next sample is stored one by one
            const int sm = tdiv(f, a.inv_TPQ), rem = f - sm * a.TPQ;
            if (rem + 4 <= a.TPQ) {
                if (f < a.npos && b0 + sm < a.N) tile_put4<DT>(y, ((int64_t)(b0 + sm) * a.D + d) * PQ + rem, v, relu, codes, rq, 4);
                return;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int smj = tdiv(f + j, a.inv_TPQ), remj = f + j - smj * a.TPQ;
                if (f + j < a.npos && b0 + smj < a.N)
                    tile_put4<DT>(y, ((int64_t)(b0 + smj) * a.D + d) * PQ + remj, Acc{v[j], v[j], v[j], v[j]}, relu, codes, rq, 1);
            }
        }
    };
    const int waves1 = 1 << (lwm + lwn);                 // waves of one group
    const int w1 = wave & (waves1 - 1);
    if (KG == 2) {
        // the second group hands its sums to the first, a lane's own 16 bytes per block
        lds_barrier();
        Acc* ex = reinterpret_cast<Acc*>(lds) + w1 * (MW * NW * 64) + lane;
        if (kgrp == 1) {
#pragma unroll
            for (int m = 0; m < MW; ++m)
#pragma unroll
                for (int i = 0; i < NW; ++i) ex[(m * NW + i) * 64] = acc[m][i];
        }
        lds_barrier();
        if (kgrp == 0) {
#pragma unroll
            for (int m = 0; m < MW; ++m)
#pragma unroll
                for (int i = 0; i < NW; ++i) acc[m][i] += ex[(m * NW + i) * 64];
        }
    }
    if (KG > 2) {
        // all groups put their sums into LDS; block b of the wave tile is added up (in the order of the groups) and
        // stored by group b mod KG
        lds_barrier();
        Acc* ex = reinterpret_cast<Acc*>(lds) + lane;
#pragma unroll
        for (int m = 0; m < MW; ++m)
#pragma unroll
            for (int i = 0; i < NW; ++i) ex[((kgrp * waves1 + w1) * (MW * NW) + m * NW + i) * 64] = acc[m][i];
        lds_barrier();
        constexpr int BPW = (MW * NW + 3) / 4;               // blocks per wave, at most
#pragma unroll
        for (int t = 0; t < BPW; ++t) {
            const int b = kgrp + t * KG;
            if (b < MW * NW) {
                Acc s = ex[(w1 * (MW * NW) + b) * 64];
                for (int g = 1; g < KG; ++g) s += ex[((g * waves1 + w1) * (MW * NW) + b) * 64];
                acc[t / NW][t % NW] = s;
            }
        }
        if (!(a.bits & 8)) {
#pragma unroll
            for (int t = 0; t < BPW; ++t) {
                const int b = kgrp + t * KG;
                if (b < MW * NW) put(b / NW, b % NW, acc[t / NW][t % NW], multiplier(b / NW));
            }
            return;
        }
    } else if (!(a.bits & 8)) {
        if (kgrp > 0) return;
#pragma unroll
        for (int m = 0; m < MW; ++m) {
            const float rq = multiplier(m);
#pragma unroll
            for (int i = 0; i < NW; ++i) put(m, i, acc[m][i], rq);
        }
        return;
    }

    // ---------------------------------------------------------------- fused epilogue with pooling: the sums as
    // [output channel][tile position] in LDS, then every thread finishes elements of y -- the maximum over
    // its 2 x 2 window, ReLU, and the store as the layer's type or, requantised, as an 8-bit code
    lds_barrier();
    A* ex = reinterpret_cast<A*>(lds);
    auto give = [&](int m, int i, const Acc& v) {
        *reinterpret_cast<Acc*>(ex + ((wm * MW + m) * 16 + n16) * a.epi_pitch + (wn * NW + i) * 16 + 4 * kg) = v;
    };
    if (KG > 2) {
        constexpr int BPW = (MW * NW + 3) / 4;
#pragma unroll
        for (int t = 0; t < BPW; ++t) {
            const int b = kgrp + t * KG;
            if (b < MW * NW) give(b / NW, b % NW, acc[t / NW][t % NW]);
        }
    } else if (kgrp == 0) {
#pragma unroll
        for (int m = 0; m < MW; ++m)
#pragma unroll
            for (int i = 0; i < NW; ++i) give(m, i, acc[m][i]);
    }
    if constexpr (kIntActs<DT>) {
        // the multipliers behind the rows (a row is 4 words longer than its sums): by the first wave that holds the row's channels
        if (kgrp == 0 && wn == 0 && kg == 0) {
#pragma unroll
            for (int m = 0; m < MW; ++m) ex[((wm * MW + m) * 16 + n16) * a.epi_pitch + a.epi_pitch - 4] = __float_as_int(rqs[m]);
        }
    }
    lds_barrier();
    // One element = V neighbouring outputs of a row (4 where the rows allow it).  A thread keeps to one element of the
    // tile (decoded once) and walks over the output channels; the threads lie as (channel group,
    // element) with the elements a power of two wide, so that small tiles still use every thread.
    auto pool = [&](auto vtag) {
        constexpr int V = decltype(vtag)::value;
        const int TPo = a.TP / 2, Qe = a.Qo / V;             // output rows of y per tile (TP is even, or the whole plane); elements per row
        const int per_s = TPo * Qe, per_d = a.NS * per_s;
        const float inv_per_s = __builtin_amdgcn_rcpf((float)max(per_s, 1)), inv_Qe = __builtin_amdgcn_rcpf((float)Qe);
        const int prow0 = p0 / 2;
        int pw2 = 1;
        while (pw2 < per_d && pw2 < NT) pw2 <<= 1;
        const int dgroups = NT / pw2;
        const int o_first = tid & (pw2 - 1), dg = tid / pw2;
        for (int o = o_first; o < per_d; o += pw2) {
            const int sm = tdiv(o, inv_per_s);
            const int r2 = o - sm * per_s;
            const int tpo = tdiv(r2, inv_Qe);
            const int tqo = (r2 - tpo * Qe) * V;
            if (b0 + sm >= a.N || prow0 + tpo >= a.Po) continue;
            const A* src = ex + sm * a.TPQ + (tpo * 2) * a.Q + tqo * 2;
            const int64_t off0 = (((int64_t)(b0 + sm) * a.D) * a.Po + prow0 + tpo) * a.Qo + tqo;
            const int64_t dstride = (int64_t)a.Po * a.Qo;
            const int dend = min(a.DB, a.D - db * a.DB);
            for (int dl = dg; dl < dend; dl += dgroups) {
                const int d = db * a.DB + dl;
                const A* sp = src + dl * a.epi_pitch;
                float rq = 0.0f;
                if constexpr (kIntActs<DT>) rq = __int_as_float(ex[dl * a.epi_pitch + a.epi_pitch - 4]);
                if constexpr (V == 4) {
                    const Acc u0 = *reinterpret_cast<const Acc*>(sp), u1 = *reinterpret_cast<const Acc*>(sp + 4);
                    const Acc w0 = *reinterpret_cast<const Acc*>(sp + a.Q), w1_ = *reinterpret_cast<const Acc*>(sp + a.Q + 4);
                    auto most = [](A p, A q, A r, A s) { return tile_max(tile_max(p, q), tile_max(r, s)); };
                    const Acc v = {most(u0[0], u0[1], w0[0], w0[1]), most(u0[2], u0[3], w0[2], w0[3]),
                                   most(u1[0], u1[1], w1_[0], w1_[1]), most(u1[2], u1[3], w1_[2], w1_[3])};
                    tile_put4<DT>(y, off0 + d * dstride, v, relu, codes, rq, 4);
                } else {
                    const A v = tile_max(tile_max(sp[0], sp[1]), tile_max(sp[a.Q], sp[a.Q + 1]));
                    tile_put4<DT>(y, off0 + d * dstride, Acc{v, v, v, v}, relu, codes, rq, 1);
                }
            }
        }
    };
    // (four outputs read 8 neighbouring sums of two rows, as 16-byte words)
    if (a.Qo % 4 == 0 && a.Q % 4 == 0) pool(std::integral_constant<int, 4>{});
    else pool(std::integral_constant<int, 1>{});
}

template <sc_dtype_t DT, int MW, int NW, int LEPV, bool WIDE>
static sc_status_t launch_tile_one(const Plan& p, const TileArgs& a, const void* x, void* y, int grid, hipStream_t stream)
{
    using X = typename Types<DT>::X;
    using Y = typename Types<DT>::Y;
    auto kernel = &mfma_tile_kernel<DT, MW, NW, LEPV, WIDE>;
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [&] {
        attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes);
    });
    if (attr_err != hipSuccess) return SC_ERR_HIP;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(p.mg.waves * 64), p.mg.lds_bytes, stream, static_cast<const X*>(x),
                       static_cast<Y*>(y), reinterpret_cast<const uint4w*>(p.d_wfrag), a);
    return hipGetLastError() == hipSuccess ? SC_OK : SC_ERR_HIP;
}

template <sc_dtype_t DT, int LEPV, bool WIDE = false>
static sc_status_t launch_tile_typed(const Plan& p, const TileArgs& a, const void* x, void* y, int grid, hipStream_t stream)
{
    switch (p.mg.MW * 10 + p.mg.NW) {
        case 11: return launch_tile_one<DT, 1, 1, LEPV, WIDE>(p, a, x, y, grid, stream);
        case 12: return launch_tile_one<DT, 1, 2, LEPV, WIDE>(p, a, x, y, grid, stream);
        case 14: return launch_tile_one<DT, 1, 4, LEPV, WIDE>(p, a, x, y, grid, stream);
        case 17: return launch_tile_one<DT, 1, 7, LEPV, WIDE>(p, a, x, y, grid, stream);
        case 18: return launch_tile_one<DT, 1, 8, LEPV, WIDE>(p, a, x, y, grid, stream);
        case 21: return launch_tile_one<DT, 2, 1, LEPV, WIDE>(p, a, x, y, grid, stream);
        case 22: return launch_tile_one<DT, 2, 2, LEPV, WIDE>(p, a, x, y, grid, stream);
        case 24: return launch_tile_one<DT, 2, 4, LEPV, WIDE>(p, a, x, y, grid, stream);
        case 27: return launch_tile_one<DT, 2, 7, LEPV, WIDE>(p, a, x, y, grid, stream);
        case 28: return launch_tile_one<DT, 2, 8, LEPV, WIDE>(p, a, x, y, grid, stream);
        case 41: return launch_tile_one<DT, 4, 1, LEPV, WIDE>(p, a, x, y, grid, stream);
        case 42: return launch_tile_one<DT, 4, 2, LEPV, WIDE>(p, a, x, y, grid, stream);
        case 44: return launch_tile_one<DT, 4, 4, LEPV, WIDE>(p, a, x, y, grid, stream);
    }
    return SC_ERR_UNSUPPORTED;
}

}  // namespace sc
