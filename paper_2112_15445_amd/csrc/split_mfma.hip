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

#include "sc_staging.h"
#include "split_kernel.h"

namespace sc {

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
    if ((WM != 1 && WM != 2 && WM != 4) || DB % (16 * WM)) return false;
    // groups that split the contraction: one or two of four waves, in the pipelined form two or four of eight waves in all
    if (PW ? (KG != 2 && KG != 4) || WM > 8 / KG : KG != 1 && KG != 2) return false;
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
    const int nb = (g.npos + 15) / 16, wn = (PW ? 8 / KG : 4) / WM, nw = (nb + wn - 1) / wn;
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
    if (PW && (PW != 4 || KS != 1 || g.MW * g.NW > 8)) return false;
    g.PW = PW;
    int64_t lds = 3ll * g.bufsz * (PW && g.nchunks > 1 ? 2 : 1);
    // (the groups hand on their sums: a wave those of the blocks that it does not store)
    if (KG >= 2) lds = std::max<int64_t>(lds, (int64_t)g.MW * g.NW * (8 / KG) * (KG - 1) * 1024);
    if (lds > lds_budget || lds > kMaxLdsBytes) return false;
    g.lds_bytes = (int)lds;
    // Columns per staging load, 4, 2 or 1 (an instruction count of a block: its loads and address; for each column 44 to split it and
    // three LDS writes).  Loads as wide as row length and pointer allow, the rule before, read rows of 7 and 31 values one at a time: see
    // split_kernel.h.
    g.flat = g.Ws == L.W && L.pad_w == 0 ? 1 : 0;
    const int64_t row = std::max(0, std::min(L.W, g.Ws - L.pad_w));
    const int64_t least = g.flat ? least_staged_rows(L.H, g.Hs, (int64_t)g.TP * L.stride_h, L.pad_h, g.tiles_p) : 1;
    g.lepv = load_columns(2, 40, 64, (int64_t)(g.CC / 8) * g.NS, PW ? 256 : 256 * KG, g.flat ? 1 : g.Hs, g.flat ? g.Hs * row : row, least * row);
    *out = g;
    return true;
}

int split_grid_size(const MfmaGeom& g, int N) { return ((N + g.NS - 1) / g.NS) * g.tiles_p * g.ndb * g.DL; }

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
    a.gq = (int)grid >> 3; a.gr = (int)grid & 7;
    a.tiles_p = g.tiles_p; a.inv_tiles_p = 1.0f / (float)g.tiles_p;
    a.NS = g.NS; a.N = N; a.TP = g.TP; a.s_h = p.L.stride_h; a.s_w = p.L.stride_w; a.pad_h = p.L.pad_h; a.pad_w = p.L.pad_w;
    a.H = p.L.H; a.Hs = g.Hs; a.W = p.L.W; a.Ws = g.Ws; a.npos1 = g.Hs * g.Ws; a.CC = g.CC; a.C = p.L.C;
    a.wcols = std::max(0, std::min(p.L.W, g.Ws - p.L.pad_w));
    a.cps = (g.nchunks + g.DL - 1) / g.DL; a.nchunks = g.nchunks;
    a.plane4 = (unsigned)(p.L.H * p.L.W) * 4u;
    a.pitch = g.pitch; a.bufsz = g.bufsz; a.npos_s = g.npos_s;
    a.DB = g.DB; a.RS = p.L.R * p.L.S; a.NCB = g.NCB; a.S = p.L.S; a.cbs_last = g.NCB - (g.nchunks - 1) * (g.CC / 32);
    a.npos = g.npos; a.TPQ = g.TP * p.Q; a.Q = p.Q;
    a.inv_TPQ = 1.0f / (float)a.TPQ; a.inv_Q = 1.0f / (float)p.Q; a.inv_npos1 = 1.0f / (float)a.npos1; a.inv_Ws = 1.0f / (float)g.Ws;
    a.P = p.P; a.D = p.L.D;
    a.floor = 2u * float_bits(p.split_floor) + (1u << 24);
    // Order of the workgroups by what an XCD reads into its L2: with the tile outermost all weights and an eighth of the input,
    // else its share of the weights and (of the chunks its workgroups take) of the input
    const int ntiles = ((N + g.NS - 1) / g.NS) * g.tiles_p;
    const double w = (double)split_weight_bytes(p), xin = (double)N * p.L.C * p.L.H * p.L.W * 4.0, combos = (double)g.ndb * g.DL;
    const bool wmajor = w / std::min(8.0, combos) + xin / g.DL * std::min(1.0, combos / 8.0) < w + xin / 8.0;
    a.inner = wmajor ? ntiles : g.ndb; a.inner2 = wmajor ? g.ndb : g.DL;
    a.inv_inner = 1.0f / (float)a.inner; a.inv_inner2 = 1.0f / (float)a.inner2;
    a.bits = (wmajor ? 1 : 0) | (g.flat ? 2 : 0) | (p.L.pad_h || p.L.pad_w ? 4 : 0) | (g.DL > 1 ? 8 : 0) | __builtin_ctz(g.WM) << 4;
    const SplitTable tab{static_cast<const float*>(p.d_theta), p.d_col, p.d_len, p.n};
    using Launch = sc_status_t (*)(const Plan&, const SplitArgs&, const SplitTable&, const void*, void*, int, hipStream_t);
    static const Launch kernels[4][3] = {{launch_split_one_1, launch_split_one_2, launch_split_one_4},
                                         {launch_split_two_1, launch_split_two_2, launch_split_two_4},
                                         {launch_split_pipe2_1, launch_split_pipe2_2, launch_split_pipe2_4},
                                         {launch_split_pipe4_1, launch_split_pipe4_2, launch_split_pipe4_4}};
    if (g.DL > 1) {
        const sc_status_t st = launch_clear(y, (int64_t)N * p.L.D * p.P * p.Q, stream);
        if (st != SC_OK) return st;
    }
    return kernels[g.PW ? __builtin_ctz(g.KG) + 1 : g.KG - 1][g.lepv](p, a, tab, x, y, (int)grid, stream);
}

}  // namespace sc
