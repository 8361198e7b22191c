// Plan construction, validation, the offset-stretching pass, tuning and dispatch of the C ABI.
//
// Follows the paper's section "Convolution operation using a sparse operation on GPGPU": CSR rows
// are output channels, rows are padded to one common stored count (the "standardised sparse level"),
// and the column indices are replaced once, ahead of time, by offsets into the padded input.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <numeric>
#include <string>
#include <unordered_set>

#include "sc_internal.h"

namespace sc {

static bool is_codebook(sc_dtype_t dt) { return dt == SC_CB4_I8 || dt == SC_CB4_F16; }   // 4-bit indices
static int codebook_bytes(sc_dtype_t dt) { return dt == SC_CB4_F16 ? 32 : 16; }
int elem_size_x(sc_dtype_t dt) { return dt == SC_F32 ? 4 : (dt == SC_F16 || dt == SC_CB4_F16) ? 2 : 1; }
int elem_size_y(sc_dtype_t dt) { return (dt == SC_F16 || dt == SC_CB4_F16) ? 2 : 4; }
// bytes of one weight as the caller passes it (clustered variants: one index per byte)
static int elem_size_w_native(sc_dtype_t dt) { return dt == SC_F32 ? 4 : dt == SC_F16 ? 2 : 1; }

// ------------------------------------------------------------------------------------------------
// Offset-stretching pass.  One thread per stored entry: decode the column into its filter tap
// (c, r, s) and emit the flat offset for a layout described by pitches.  With nsh = nsw = 1,
// chan_pitch = Hp*Wp, row_pitch = Wp and scale = 1 this is the canonical offset into one padded
// sample, c*Hp*Wp + r*Wp + s; the slab kernel uses the same pass with its LDS tile pitches, its
// stride-phase split and scale = bytes per element.
// ------------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
stretch_kernel(const int32_t* __restrict__ col, int32_t* __restrict__ lam, int64_t count, int R,
               int S, int nsh, int nsw, int s_h, int s_w, int chan_pitch, int sub_pitch,
               int row_pitch, int scale, int chan_mod)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    // bit 31 of a column marks a zero-valued filler entry of the 4-bit codebook variant (a 4-bit
    // index cannot say "zero"); it is carried over to the offset so the kernel can zero the weight
    const int flag = col[i] & (int)0x80000000;
    const int k = col[i] & 0x7fffffff;
    const int cfull = k / (R * S);
    const int rs = k - cfull * (R * S);
    const int c = chan_mod > 0 ? cfull % chan_mod : cfull;  // channel within its LDS chunk
    const int r = rs / S;
    const int s = rs - r * S;
    const int phase = (r % nsh) * nsw + (s % nsw);
    // when a stride exceeds the filter extent only phase 0 exists along that axis and r / s_h is 0
    lam[i] = ((c * chan_pitch + phase * sub_pitch + (r / s_h) * row_pitch + (s / s_w)) * scale) | flag;
}

sc_status_t launch_stretch(const Plan& p, int32_t* d_out, int nsh, int nsw, int s_h, int s_w,
                           int chan_pitch, int sub_pitch, int row_pitch, int scale, int chan_mod,
                           hipStream_t stream)
{
    const int64_t count = (int64_t)p.L.D * p.n;
    if (count == 0) return SC_OK;
    const unsigned blocks = (unsigned)((count + 255) / 256);
    hipLaunchKernelGGL(stretch_kernel, dim3(blocks), dim3(256), 0, stream, p.d_col, d_out, count,
                       p.L.R, p.L.S, nsh, nsw, s_h, s_w, chan_pitch, sub_pitch, row_pitch, scale, chan_mod);
    return hipGetLastError() == hipSuccess ? SC_OK : SC_ERR_HIP;
}

// ------------------------------------------------------------------------------------------------
// Tuning resolution: fill heuristic defaults, derive the slab geometry, check that it fits.
// ------------------------------------------------------------------------------------------------
static bool is_pointwise(const sc_layer_t& L)
{
    return L.R == 1 && L.S == 1 && L.stride_h == 1 && L.stride_w == 1 && L.pad_h == 0 && L.pad_w == 0;
}

static int round_up(int v, int m) { return (v + m - 1) / m * m; }

// Derive the slab geometry for tile (TP, TQ); returns false if it cannot run.
static bool slab_geometry(const Plan& p, int TP, int TQ, int wg_threads, int wsrc, int pipeline, int producers,
                          int chunk_c, int tile_d, int samples, int pack, int lds_budget, SlabGeom* g, int buffers = 0)
{
    const sc_layer_t& L = p.L;
    SlabGeom o{};
    const bool pw = is_pointwise(L);
    o.Hf = pw ? 1 : L.H;
    o.Wf = pw ? L.H * L.W : L.W;
    o.Pf = pw ? 1 : p.P;
    o.Qf = pw ? p.P * p.Q : p.Q;
    if (TP < 1 || TQ < 1) return false;
    o.TP = std::min(TP, o.Pf);
    o.TQ = std::min(TQ, o.Qf);
    o.tiles_p = (o.Pf + o.TP - 1) / o.TP;
    o.tiles_q = (o.Qf + o.TQ - 1) / o.TQ;
    o.nsh = std::min(L.R, L.stride_h);
    o.nsw = std::min(L.S, L.stride_w);
    o.SR = o.TP + (L.R - 1) / L.stride_h;
    o.Qs = o.TQ + (L.S - 1) / L.stride_w;
    o.sub_pitch = o.SR * o.Qs;
    o.chan_pitch = o.nsh * o.nsw * o.sub_pitch;
    o.F = o.TP * o.Qs;
    o.fs = 1;
    if (samples > 1 && pack && pack != 3) {
        // small planes of a pointwise layer: the planes of `samples` consecutive samples laid end to
        // end form the tile's position axis (channel-major in LDS like any pointwise tile), so that
        // the lanes and the wide words of the packed forms fill up where one plane is smaller than
        // a wave.  The channel pitch is a whole number of words: no shifted images.
        if (!pw || pipeline != 0 || chunk_c <= 0 || wsrc != 1 || o.tiles_q != 1 || samples > 16) return false;
        const int words = (pack == 2 ? 16 : 4) / p.ex;
        o.fs = samples;
        o.F = samples * o.Qf;
        o.Qs = o.F;
        o.sub_pitch = o.chan_pitch = round_up(o.F, words);
        if ((int64_t)samples * L.C * o.Wf >= (1ll << 31) || (int64_t)samples * L.D * o.Qf >= (1ll << 31)) return false;
        samples = 1;
    }
    if (o.F > kWave * kMaxVpt) return false;
    o.vpt = (o.F + kWave - 1) / kWave;
    o.pack = 1;
    o.si = 0;
    if (pack == 3) {
        // samples interleaved: an LDS word holds the same position of 4 (32-bit floats, 8-bit
        // integers) or 8 (16-bit floats) consecutive samples, so every offset is a whole word on
        // any layer shape; chunked one-shot form, weights by scalar loads
        if (pipeline != 0 || chunk_c <= 0 || wsrc != 1) return false;
        if (p.dtype != SC_F32 && p.dtype != SC_F16 && p.dtype != SC_I8) return false;
        o.si = 1;
        o.pack = p.dtype == SC_I8 ? 4 : 16 / p.ex;
        if (o.vpt * o.pack > 8) return false;
        // small planes: `samples` such groups per workgroup, the lanes numbered over (group, position)
        // -- a 4 x 4 plane with its halo column fills 24 of 64 lanes, two groups of it 48
        o.sg = 1;
        if (samples > 1) {
            if (o.vpt != 1 || samples > 8 || samples * o.F > kWave) return false;
            o.sg = samples;
            samples = 1;
        }
    } else if (pack) {
        // packed positions: chunked forms, one sample per workgroup; a lane owns the adjacent
        // positions of one 32-bit word (pack = 1: 16- or 8-bit activations) or of one 128-bit word
        // (pack = 2: 32- or 16-bit activations), at most 8 positions
        // (128-bit words also in the producer/consumer kernel without channel chunks)
        // and in the full-channel one-shot kernel on pointwise layers whose tiles are whole words)
        if (samples > 1 || (chunk_c <= 0 && !(pack == 2 && wsrc == 1 && (pipeline == 1 || (pipeline == 0 && pw)))))
            return false;
        if (pack == 1 && p.dtype != SC_F16 && p.dtype != SC_I8) return false;
        if (pack == 2 && p.dtype != SC_F32 && p.dtype != SC_F16) return false;
        o.pack = (pack == 2 ? 16 : 4) / p.ex;
        o.vpt = (o.F + kWave * o.pack - 1) / (kWave * o.pack);
        if (o.vpt * o.pack > 8) return false;
    }
    o.nwaves = wg_threads / kWave;
    o.CC = chunk_c > 0 ? std::min(chunk_c, L.C) : L.C;
    o.nchunks = (L.C + o.CC - 1) / o.CC;
    o.DTW = (chunk_c > 0 && tile_d > 0) ? std::min(tile_d, L.D) : L.D;
    o.ndt = (L.D + o.DTW - 1) / o.DTW;
    o.rpw = 0;
    if (chunk_c > 0) {
        // chunked form: pointwise layers, pipelined, weights by scalar loads; every consumer wave
        // keeps the accumulators of its rows in registers across the chunks of a tile
        // (pipeline 1 / 2: pointwise layers only; the one-shot chunked form takes any layer)
        // (weights by scalar loads; the one-shot chunked form also takes them one entry per lane)
        if ((!pw && pipeline >= 1) || !(wsrc == 1 || (wsrc == 3 && pipeline == 0 && !pack)) ||
            is_codebook(p.dtype) || p.n == 0) return false;
        const int ncons = o.nwaves - (pipeline == 1 ? producers : 0);
        if (ncons < 1) return false;
        if (pipeline != 1 && o.vpt * o.pack > (pack ? 8 : 4)) return false;
        o.rpw = (o.DTW + ncons - 1) / ncons;
        if (o.rpw > kMaxRowsPerWave) return false;
    }
    // several samples per workgroup: chunked one-shot form, tiles of at most one wave of positions
    o.ns = 1;
    if (samples > 1) {
        if (pipeline != 0 || chunk_c <= 0 || o.vpt != 1 || samples > 4) return false;
        o.ns = samples;
    }
    int64_t slab = (int64_t)o.ns * (o.si ? o.pack * o.sg : 1) * o.CC * o.chan_pitch * p.ex + (int64_t)kWave * o.vpt * o.pack * p.ex;
    // packed positions read aligned 32-bit words only (unaligned LDS reads are several times
    // slower): unless every lambda is a whole number of words (pointwise layer, even channel
    // pitch), LDS holds `pack` images of the chunk, image s shifted by s elements, and an entry
    // with lambda = s (mod pack) reads image s at lambda - s
    o.copies = 1;
    if (o.pack > 1 && !o.si && pipeline == 0 && !(pw && o.chan_pitch % o.pack == 0)) o.copies = o.pack;
    slab = (int64_t)o.copies * round_up((int)std::min<int64_t>(slab, kMaxLdsBytes), 16);
    if (slab > lds_budget) return false;
    o.slab_bytes = round_up((int)slab, 16);
    o.copy_bytes = o.slab_bytes / o.copies;
    // weight stage: as many (theta, lambda) pairs as the budget allows, within [512, 4096]
    const int64_t total = (int64_t)L.D * p.n;
    int64_t cap = (lds_budget - o.slab_bytes - 64 - round_up(o.chan_pitch * 4, 16)) / 8;
    cap = std::min<int64_t>(cap, 4096);
    cap = std::min<int64_t>(cap, std::max<int64_t>(total, 1));
    if (wsrc != 0) cap = 0;  // weights straight from global memory: no weight stage in LDS
    else if (cap < std::min<int64_t>(std::max<int64_t>(total, 1), 512)) return false;
    o.wcap = (int)cap;
    if (p.n == 0 || wsrc != 0) {
        o.DS = std::min(L.D, o.nwaves);
        o.JC = 0;
    } else if ((int64_t)p.n * std::min(o.nwaves, L.D) <= o.wcap) {
        o.JC = p.n;                       // whole rows per stage
        o.DS = std::min(L.D, o.wcap / p.n);
    } else {
        o.DS = std::min(L.D, o.nwaves);   // one row per wave, rows cut into chunks
        o.JC = std::max(1, o.wcap / o.DS);
    }
    // the one-shot forms keep a table of chan_pitch plane offsets behind the slab (chunked form) or
    // behind the weight stage and the codebook (full-channel form)
    o.lds_bytes = o.slab_bytes + o.wcap * 8 + 64 + round_up(o.chan_pitch * 4, 16);
    if (pipeline == 0 && chunk_c > 0) o.lds_bytes = o.slab_bytes + round_up(o.chan_pitch * 4, 16) + 64;
    o.nbuf = 2;
    if (pipeline == 1) {
        // two tile buffers, no weight stage; only for pointwise layers whose rows can be copied
        // 16 bytes at a time, and the workgroup needs consumer waves besides the producers
        // (with channel chunks: optionally producers + 1 buffers, a producer wave per chunk in flight)
        if (!pw || wsrc == 0 || o.nwaves < 8) return false;
        if (buffers > 2) {
            if (chunk_c <= 0 || buffers != producers + 1 || buffers > 5) return false;
            o.nbuf = buffers;
        }
        o.lds_bytes = o.nbuf * o.slab_bytes;
    } else if (buffers > 2) {
        return false;
    }
    // (a caller whose x is not aligned for the direct-to-LDS copies is served by the one-shot kernel
    // with this same allocation: it must also hold that kernel's tile plus its offset table)
    const int one_shot_bytes = o.slab_bytes + 64 + round_up(o.chan_pitch * 4, 16);
    if (pipeline == 2) {
        // symmetric form: two tile buffers, scalar-load weights, at least one stored entry per row
        if (!pw || wsrc != 1 || p.n == 0) return false;
        o.lds_bytes = 2 * o.slab_bytes;
    }
    if (pipeline >= 1 && chunk_c <= 0) o.lds_bytes = std::max(o.lds_bytes, one_shot_bytes);
    if (o.lds_bytes > lds_budget || o.lds_bytes > kMaxLdsBytes) return false;
    // 16-byte staging needs every tile row start and the plane pitch to be 16-byte aligned
    const int epv = 16 / p.ex;
    o.vec = (pw && (o.Wf % epv == 0) && (o.TQ % epv == 0)) ? 1 : 0;
    // direct-to-LDS copies: 16 bytes per lane for such rows, else 4 bytes per lane when the rows are
    // at least 4-byte aligned (only the symmetric kernels take that form)
    const int epd = std::max(1, 4 / p.ex);
    o.dmab = o.vec ? 16 : ((pw && (o.Wf % epd == 0) && (o.TQ % epd == 0)) ? 4 : 0);
    if (pipeline == 1 && !o.vec) return false;
    if (pipeline == 2 && o.dmab == 0) return false;
    if (pack && pipeline >= 1 && o.dmab == 0) return false;      // whole words per row and tile
    if (pack == 2 && pipeline >= 1 && o.dmab != 16) return false;
    if (pack == 2 && pipeline == 0 && chunk_c <= 0 && (o.chan_pitch % o.pack != 0 || o.Wf % o.pack != 0)) return false;
    o.inv_chan_pitch = 1.0f / (float)o.chan_pitch;
    o.inv_sub_pitch = 1.0f / (float)o.sub_pitch;
    o.inv_Qs = 1.0f / (float)o.Qs;
    *g = o;
    return true;
}

// DENSE variant: fill the fields left 0 and derive the geometry.
static sc_status_t resolve_dense(const Plan& p, sc_tuning_t t, sc_tuning_t* out, MfmaGeom* mgeom)
{
    const sc_layer_t& L = p.L;
    if (p.dtype == SC_F32 || p.has_dup || p.n == 0) return SC_ERR_UNSUPPORTED;
    // (eight waves that split the contraction four ways and more hand on up to 128 KB of sums through LDS)
    if (t.wg_per_cu == 0) t.wg_per_cu = t.buffers == 8 || (t.buffers == 4 && t.wg_threads == 512) ? 1 : 2;
    if (t.wg_per_cu < 1 || t.wg_per_cu > 8) return SC_ERR_UNSUPPORTED;
    if (t.tile_p < 0 || t.sub_batch < 0 || t.chunk_c < 0 || t.tile_d < 0) return SC_ERR_UNSUPPORTED;
    if (t.wsrc || t.ragged || t.pack || t.tile_q) return SC_ERR_UNSUPPORTED;
    // split_n = 2 .. 16: the workgroup walks over that many blocks of tile_d output channels, the tile resident in LDS
    if (t.split_n < 0 || t.split_n > 16) return SC_ERR_UNSUPPORTED;
    const int DL = std::max(1, t.split_n);
    // stage_rows = 1: pointwise layers staged in their natural layout (pipelined: by direct-to-LDS copies)
    if (t.stage_rows != 0 && t.stage_rows != 1) return SC_ERR_UNSUPPORTED;
    if (t.stage_rows && !is_pointwise(L)) return SC_ERR_UNSUPPORTED;
    const int nat = t.stage_rows;
    // pipeline = 1: the chunks are staged by `producers` waves of their own (1 .. 4, default 2), one chunk ahead
    if (t.pipeline != 0 && t.pipeline != 1) return SC_ERR_UNSUPPORTED;
    if (t.producers < 0 || t.producers > 4 || (t.producers && !t.pipeline)) return SC_ERR_UNSUPPORTED;
    const int PW = t.pipeline ? (t.producers ? t.producers : 2) : 0;
    const int budget = kMaxLdsBytes / t.wg_per_cu;
    const int CB = mfma_chan_block(p.dtype);
    // 256 threads: four waves; 512: two groups of four that split the steps of the contraction
    if (t.wg_threads != 0 && t.wg_threads != 256 && t.wg_threads != 512) return SC_ERR_UNSUPPORTED;
    // (by default four waves; eight groups of waves need eight)
    const int waves = t.wg_threads == 512 || (t.wg_threads == 0 && t.buffers == 8) ? 8 : 4;
    // buffers = 1, 2, 4 or 8: that many groups of waves split the contraction (one-shot form on the transposed tile)
    if (t.buffers != 0 && t.buffers != 1 && t.buffers != 2 && t.buffers != 4 && t.buffers != 8) return SC_ERR_UNSUPPORTED;
    if (t.buffers && (t.pipeline || nat || DL > 1)) return SC_ERR_UNSUPPORTED;
    const int KG = t.buffers ? t.buffers : waves / 4;
    if (t.waves_m != 0 && t.waves_m != 1 && t.waves_m != 2 && t.waves_m != 4) return SC_ERR_UNSUPPORTED;
    // (more groups leave fewer waves to a group: the default tile is what those can own, 64 channels a wave, or 32
    // where a wave of 64, which holds 64 positions, could not take the least tile: a row of outputs, two under pooling)
    const int group = waves / KG;
    if (group < 1) return SC_ERR_UNSUPPORTED;
    int DB = t.tile_d;
    if (DB == 0) DB = std::min(L.D > 64 ? 128 : (L.D > 32 ? 64 : (L.D > 16 ? 32 : 16)), (p.Q * (p.epi.pool ? 2 : 1) > 64 ? 32 : 64) * group);
    // waves along the output channels: by default as many as still leave every wave 32 channels
    // (two 16-row blocks), so that the weights, which every wave fetches for itself from L2, are
    // fetched by few waves each
    int WM = t.waves_m;
    if (WM == 0) WM = std::min(DB >= 128 ? 4 : (DB >= 64 ? 2 : 1), group);
    if (DB % (16 * WM) || DB / (16 * WM) < 1 || DB / (16 * WM) > 4) return SC_ERR_UNSUPPORTED;
    const int MWv = DB / (16 * WM);
    if (waves % (WM * KG)) return SC_ERR_UNSUPPORTED;
    const int maxpos = (waves / (WM * KG)) * (MWv == 4 ? 4 : 8) * 16;    // positions the waves of a group can hold
    int TP = t.tile_p, NS = t.sub_batch;
    const bool fixed_tile = TP != 0 || NS != 0;
    if (TP == 0 && NS == 0) {
        if (p.P * p.Q <= maxpos) { TP = p.P; NS = std::max(1, std::min(16, maxpos / (p.P * p.Q))); }
        else { TP = std::max(1, maxpos / p.Q); NS = 1; }
    }
    if (TP == 0) TP = p.P;
    if (NS == 0) NS = 1;
    MfmaGeom g{};
    for (;;) {
        bool ok = false;
        if (t.chunk_c) ok = mfma_geometry(p, TP, NS, t.chunk_c, DB, WM, budget, &g, waves, KG, PW, nat, DL);
        else
            // (one-shot: the largest chunk that fits; pipelined: small chunks are the point -- two blocks)
            for (int cc = PW ? std::min(2 * CB, (L.C + CB - 1) / CB * CB) : (L.C + CB - 1) / CB * CB; cc >= CB && !ok; cc -= CB)
                ok = mfma_geometry(p, TP, NS, cc, DB, WM, budget, &g, waves, KG, PW, nat, DL);
        if (ok) break;
        if (fixed_tile) return SC_ERR_UNSUPPORTED;
        // heuristic tile too large for LDS or for the waves: fewer samples, then fewer rows
        if (NS > 1) NS /= 2;
        else if (TP > 1) TP = (TP + 1) / 2;
        else return SC_ERR_UNSUPPORTED;
    }
    sc_tuning_t r{};
    r.variant = SC_VARIANT_DENSE;
    r.wg_threads = 64 * waves;
    r.buffers = KG == waves / 4 ? 0 : KG;
    r.tile_p = g.TP;
    r.sub_batch = g.NS;
    r.chunk_c = g.CC;
    r.tile_d = g.DB;
    r.waves_m = g.WM;
    r.wg_per_cu = t.wg_per_cu;
    r.pipeline = PW ? 1 : 0;
    r.producers = PW;
    r.stage_rows = nat;
    r.split_n = g.DL > 1 ? g.DL : 0;
    *out = r;
    *mgeom = g;
    return SC_OK;
}

// The split form (SLAB with pipeline = 3): fill the fields left 0 and derive the geometry.
static sc_status_t resolve_split(const Plan& p, sc_tuning_t t, sc_tuning_t* out, MfmaGeom* mgeom)
{
    const sc_layer_t& L = p.L;
    if (p.dtype != SC_F32 || !p.splittable || p.has_dup || p.n == 0 || has_epilogue(p)) return SC_ERR_UNSUPPORTED;
    if (t.wsrc || t.ragged < 0 || t.ragged > 1 || t.pack || t.tile_q || t.stage_rows) return SC_ERR_UNSUPPORTED;
    // (the dense image never holds the fillers: ragged = 1 says so, the result is the same)
    if (t.producers != 0 && t.producers != 4) return SC_ERR_UNSUPPORTED;      // 4: staging waves of their own, two chunk buffers
    const int PW = t.producers;
    if (t.wg_threads != 0 && t.wg_threads != 256 && t.wg_threads != 512) return SC_ERR_UNSUPPORTED;
    // groups that split the contraction: one or two of four waves (eight by default: two per SIMD); in the pipelined form, whose
    // multiplying waves are eight, two of four or (buffers = 4) four of two
    if (t.buffers != 0 && (!PW || t.wg_threads == 256 || t.buffers != 4)) return SC_ERR_UNSUPPORTED;
    const int KG = t.buffers ? t.buffers : (t.wg_threads == 256 ? 1 : 2);
    if (t.wg_per_cu == 0) t.wg_per_cu = 1;
    if (t.wg_per_cu < 1 || t.wg_per_cu > 8) return SC_ERR_UNSUPPORTED;
    if (t.tile_p < 0 || t.sub_batch < 0 || t.chunk_c < 0 || t.tile_d < 0 || t.waves_m < 0 || t.split_n < 0) return SC_ERR_UNSUPPORTED;
    const int budget = kMaxLdsBytes / t.wg_per_cu;
    const int KS = std::max(1, t.split_n);
    const int DB = t.tile_d ? t.tile_d : (L.D > 32 ? 64 : (L.D > 16 ? 32 : 16));
    const int waves = PW ? 8 / KG : 4;                        // of one group
    const int WM = t.waves_m ? t.waves_m : std::min(waves, DB >= 64 ? 2 : 1);
    int TP = t.tile_p, NS = t.sub_batch;
    const bool fixed_tile = TP != 0 || NS != 0;
    const int maxpos = std::max(1, waves / WM) * 64;
    if (!fixed_tile) {
        if (p.P * p.Q <= maxpos) { TP = p.P; NS = std::max(1, std::min(16, maxpos / (p.P * p.Q))); }
        else { TP = std::max(1, maxpos / p.Q); NS = 1; }
    }
    if (TP == 0) TP = p.P;
    if (NS == 0) NS = 1;
    MfmaGeom g{};
    for (;;) {
        bool ok = false;
        if (t.chunk_c) ok = split_geometry(p, TP, NS, t.chunk_c, DB, WM, KG, KS, PW, budget, &g);
        else
            for (int cc = PW ? 64 : (L.C + 31) / 32 * 32; cc >= 32 && !ok; cc -= 32) ok = split_geometry(p, TP, NS, cc, DB, WM, KG, KS, PW, budget, &g);
        if (ok) break;
        if (fixed_tile) return SC_ERR_UNSUPPORTED;
        if (NS > 1) NS /= 2;
        else if (TP > 1) TP = (TP + 1) / 2;
        else return SC_ERR_UNSUPPORTED;
    }
    sc_tuning_t r{};
    r.variant = SC_VARIANT_SLAB;
    r.pipeline = 3;
    r.wg_threads = PW ? 512 : 256 * KG;
    r.buffers = KG > 2 ? KG : 0;
    r.tile_p = g.TP;
    r.sub_batch = g.NS;
    r.chunk_c = g.CC;
    r.tile_d = g.DB;
    r.waves_m = g.WM;
    r.wg_per_cu = t.wg_per_cu;
    r.producers = PW;
    r.ragged = t.ragged;
    r.split_n = KS > 1 ? KS : 0;
    *out = r;
    *mgeom = g;
    return SC_OK;
}

sc_status_t resolve_tuning(const Plan& p, const sc_tuning_t& in, sc_tuning_t* out, SlabGeom* geom, MfmaGeom* mgeom)
{
    sc_tuning_t t = in;
    const sc_layer_t& L = p.L;
    if (t.variant < SC_VARIANT_AUTO || t.variant > SC_VARIANT_DENSE) return SC_ERR_UNSUPPORTED;
    if (t.variant == SC_VARIANT_DENSE) {
        *geom = SlabGeom{};
        return resolve_dense(p, t, out, mgeom);
    }
    if (is_split(t)) {
        *geom = SlabGeom{};
        return resolve_split(p, t, out, mgeom);
    }
    *mgeom = MfmaGeom{};
    if (t.waves_m) return SC_ERR_UNSUPPORTED;
    if (t.wg_threads == 0) t.wg_threads = 256;
    if (t.wg_threads < 64 || t.wg_threads > 1024 || t.wg_threads % 64) return SC_ERR_UNSUPPORTED;
    if (t.wsrc < 0 || t.wsrc > 3) return SC_ERR_UNSUPPORTED;
    if (t.wsrc != 0 && is_codebook(p.dtype)) return SC_ERR_UNSUPPORTED;  // indices are decoded in LDS
    if (t.pipeline < 0 || t.pipeline > 2) return SC_ERR_UNSUPPORTED;
    if (t.buffers < 0 || t.buffers == 1 || t.buffers > 5) return SC_ERR_UNSUPPORTED;
    if (t.buffers == 2) t.buffers = 0;
    if (t.buffers > 2) {
        if (t.pipeline != 1 || t.chunk_c <= 0) return SC_ERR_UNSUPPORTED;
        if (t.producers == 0) t.producers = t.buffers - 1;
    }
    if (t.pipeline == 1 && t.producers == 0) t.producers = 2;
    if (t.pipeline != 1) t.producers = 0;
    if (t.chunk_c < 0 || t.tile_d < 0) return SC_ERR_UNSUPPORTED;
    if (t.chunk_c == 0) t.tile_d = 0;
    if (t.ragged < 0 || t.ragged > 1) return SC_ERR_UNSUPPORTED;
    if (t.chunk_c == 0) t.ragged = 0;
    if (t.pack < 0 || t.pack > 3) return SC_ERR_UNSUPPORTED;
    if (t.producers != 0 && t.producers != 1 && t.producers != 2 && t.producers != 4 && !(t.producers == 3 && t.buffers == 4))
        return SC_ERR_UNSUPPORTED;
    // (a fused epilogue lives in the GATHER and DENSE kernels only)
    if (has_epilogue(p) && t.variant == SC_VARIANT_SLAB) return SC_ERR_UNSUPPORTED;
    const bool want_slab = t.variant != SC_VARIANT_GATHER && !has_epilogue(p);
    if (want_slab) {
        const bool pw = is_pointwise(L);
        if (t.wg_per_cu == 0) t.wg_per_cu = t.pipeline >= 1 ? 1 : 2;
        if (t.wg_per_cu < 1 || t.wg_per_cu > 8) return SC_ERR_UNSUPPORTED;
        const int budget = kMaxLdsBytes / t.wg_per_cu;
        SlabGeom g{};
        bool ok = false;
        // sub_batch means samples per workgroup for the chunked one-shot form only
        // (with packed positions: samples laid end to end in one tile, up to 16)
        const int samples = (t.pipeline == 0 && t.chunk_c > 0) ? t.sub_batch : 0;
        if (samples < 0 || samples > (t.pack ? 16 : 4)) return SC_ERR_UNSUPPORTED;
        if (t.tile_q == 0) {
            // heuristic: widest tile that fits; pointwise layers tile the flattened plane in
            // multiples of a wave, other layers take full rows and as many of them as fit
            if (pw) {
                const int hw = L.H * L.W;
                for (int v = kMaxVpt; v >= 1 && !ok; --v) {
                    const int tq = std::min(hw, 64 * v);
                    ok = slab_geometry(p, 1, tq, t.wg_threads, t.wsrc, t.pipeline, t.producers, t.chunk_c, t.tile_d, samples, t.pack, budget, &g, t.buffers);
                }
            } else {
                for (int tp = (t.tile_p ? t.tile_p : p.P); tp >= 1 && !ok; --tp) {
                    ok = slab_geometry(p, tp, p.Q, t.wg_threads, t.wsrc, t.pipeline, t.producers, t.chunk_c, t.tile_d, samples, t.pack, budget, &g, t.buffers);
                    if (t.tile_p) break;
                }
            }
        } else {
            ok = slab_geometry(p, pw ? 1 : (t.tile_p ? t.tile_p : 1), t.tile_q, t.wg_threads, t.wsrc, t.pipeline, t.producers, t.chunk_c, t.tile_d, samples, t.pack, budget, &g, t.buffers);
        }
        // an explicit SLAB tuning with split_n > 1: the chunks of a tile are dealt to that many
        // workgroups (chunked one-shot form; fp32 and int8, whose outputs are 32-bit and can be
        // added atomically)
        int ksplit = 1;
        if (ok && in.variant == SC_VARIANT_SLAB && t.split_n > 1) {
            if (t.pipeline != 0 || t.chunk_c <= 0 || t.split_n > 16 || (p.dtype != SC_F32 && p.dtype != SC_I8) ||
                g.nchunks < t.split_n)
                return SC_ERR_UNSUPPORTED;
            ksplit = t.split_n;
        }
        if (ok) {
            t.variant = SC_VARIANT_SLAB;
            t.tile_p = g.TP;
            t.tile_q = g.TQ;
            t.sub_batch = g.ns > 1 ? g.ns : (g.fs > 1 ? g.fs : (g.sg > 1 ? g.sg : 0));
            t.split_n = ksplit > 1 ? ksplit : 0;
            g.ksplit = ksplit;
            if (t.stage_rows) {
                if (t.stage_rows != 1 || !g.si || p.dtype != SC_F32 || !slab_rows_stageable(p, g)) return SC_ERR_UNSUPPORTED;
                g.srow = 1;
            }
            if (t.pipeline >= 1) t.wg_per_cu = 1;
            if (t.chunk_c > 0) { t.chunk_c = g.CC; t.tile_d = g.DTW; }
            *out = t;
            *geom = g;
            return SC_OK;
        }
        if (t.variant == SC_VARIANT_SLAB) return SC_ERR_UNSUPPORTED;
    }
    t.variant = SC_VARIANT_GATHER;
    t.wg_threads = 256;
    if (t.sub_batch == 0) t.sub_batch = 4;
    if (t.sub_batch != 1 && t.sub_batch != 2 && t.sub_batch != 4 && t.sub_batch != 8)
        return SC_ERR_UNSUPPORTED;
    if (t.split_n == 0) t.split_n = 1;
    if (t.split_n != 1 && t.split_n != 4 && t.split_n != 16 && t.split_n != 64)
        return SC_ERR_UNSUPPORTED;
    if (has_epilogue(p) && t.split_n != 1) return SC_ERR_UNSUPPORTED;
    t.tile_p = t.tile_q = t.wg_per_cu = t.wsrc = t.pipeline = t.producers = t.chunk_c = t.tile_d = t.ragged = 0;
    if (t.pack || t.buffers || t.stage_rows) return SC_ERR_UNSUPPORTED;
    *out = t;
    *geom = SlabGeom{};
    return SC_OK;
}

// ------------------------------------------------------------------------------------------------
// The launch shape of a plan that nobody has tuned.
//
// The matrix-core tiles (DENSE; for fp32 the split form) need the same time at any sparsity, while the
// gather kernels' time grows with the entries of the unified table (fillers included: they are multiplied), D n,
// and has little to do with K = C R S.  The tile is taken where it is faster at any batch, as measured on 7700 seeded
// layers (1x1 to 7x7 and 1-D, 8 .. 2048 channels, planes of 2 .. 112, batches of 1 .. 128, 30 .. 96.5 %), both
// sides untuned (profiles/default_launch_shape_of_untuned_plans.md):
//   against the slab kernel   at least 32 output channels and 32 entries a row, a table of at least 32768 (fp32),
//                             16384 (fp16, int8) or 8192 (codebook) entries, and at least 1 weight in 12
//                             (fp32, fp16) or 24 (int8, codebook) stored, input channels counted in whole blocks: 1.0 - 400
//                             times as fast, one layer in 150 slower (0.5 - 0.95); of the fp32 layers below these lines half lose
//                             up to 5 times (1x1 64-256 at 56 x 56, batch 32, 90 %: 45 us for 26)
//   against GATHER            (the slab does not fit, or there is an epilogue) also 128 entries a row and 1
//                             weight in 16: GATHER spreads a single image over more workgroups
//   large tables              of twice as many entries, 128 or more a row: from 1 weight in 32 on, against either
//                             (1.1 - 9 times as fast; one layer in 60 slower, 0.79)
// (the fp16, int8 and codebook lines with the one-shot kernel of that time; the present one takes 0.68 of its time in the
// mean over 742 such layers of another draw, with the tile that is chosen now, and 1.03 - 1.22 of it on 16 of them)
// and the dense weights are at most 256 MB.  The tile is the one with the least estimated time of a batch of
// 32: per workgroup the largest of its matrix instructions (22 clocks each with two waves on a SIMD,
// 32 with one: measured), its weights and input through the vector L1 (64 bytes a clock) and its
// operands from LDS (128 bytes a clock), plus a fixed 8000 clocks of start and drain.  (Loads of 1 KB a wave alone reach
// 39 - 45; with 45 here the chosen tiles are no faster.)
// Four and eight groups of waves (tuning.buffers) are taken only where they are no slower at a batch of 128 either: they pay
// with small tiles, which stage the halo of the input again and again, and a batch of 32 may be too few workgroups for that to
// show (int8 3x3 283-68 stride 2 at 20 x 17, batch 128: 52 us so, 31 with one group).
// ------------------------------------------------------------------------------------------------
static bool default_dense_tuning(const Plan& p, int gather_variant, sc_tuning_t* out, MfmaGeom* mgeom)
{
    const sc_layer_t& L = p.L;
    const bool split = p.dtype == SC_F32;
    const int CB = split ? 32 : mfma_chan_block(p.dtype);
    const int64_t K = (int64_t)((L.C + CB - 1) / CB * CB) * L.R * L.S, n = p.n;      // (the tile's: whole blocks of channels)
    if (p.has_dup || (split && !p.splittable)) return false;
    const int64_t entries = split ? 32768 : (is_codebook(p.dtype) ? 8192 : 16384);
    if (L.D < 32 || n < 32 || L.D * n < entries || n * 32 < K) return false;
    if (n < 128 || L.D * n < 2 * entries) {
        if (n * (split || p.dtype == SC_F16 ? 12 : 24) < K) return false;
        if (gather_variant == SC_VARIANT_GATHER && (n < 128 || n * 16 < K)) return false;
    }
    if ((split ? split_weight_bytes(p) : mfma_weight_bytes(p)) > ((size_t)256 << 20)) return false;
    const int terms = split ? 3 : 1, products = split ? (p.split_full ? 8 : 6) : 1;
    const int64_t steps = (int64_t)L.R * L.S * ((L.C + CB - 1) / CB);
    struct Choice { double time = INFINITY, time128 = INFINITY; sc_tuning_t tuning{}; MfmaGeom geom{}; } best[2];      // tuning.buffers 0; 4 or 8
    const int layouts[][2] = {{32, 1}, {32, 2}, {64, 2}, {64, 4}, {128, 4}, {128, 2}, {64, 1}};
    for (int thr : {256, 512}) for (int kg : {0, 4, 8}) for (const auto& lw : layouts) for (int wpc : {1, 2}) for (int tile = 0; tile < 10; ++tile) {
        if (lw[0] > 32 && lw[0] >= 2 * L.D) continue;
        if ((split && kg) || (lw[0] == 64 && lw[1] == 1 && !kg)) continue;
        static const int rows[] = {1, 2, 4, 7, 8, 14};
        const int tp = tile < 6 ? rows[tile] : p.P, ns = tile < 6 ? 1 : 1 << (tile - 6);
        if (tile < 6 && tp >= p.P) continue;
        sc_tuning_t t{}, r{};
        t.variant = split ? SC_VARIANT_SLAB : SC_VARIANT_DENSE;
        t.pipeline = split ? 3 : 0;
        t.wg_threads = thr; t.tile_d = lw[0]; t.waves_m = lw[1]; t.wg_per_cu = wpc; t.tile_p = tp; t.sub_batch = ns; t.buffers = kg;
        MfmaGeom g{};
        if ((split ? resolve_split(p, t, &r, &g) : resolve_dense(p, t, &r, &g)) != SC_OK) continue;
        // (what the launch would refuse)
        if ((int64_t)g.NS * L.C * L.H * L.W >= (1ll << 29) || (int64_t)g.DB * g.npos >= (1 << 19) || g.npos_s >= (1 << 16) ||
            (int64_t)g.tiles_p * g.ndb >= (1 << 19))
            continue;
        // clocks of a batch of N.  (Workgroups that share a CU: by LDS, and on the one-shot kernel by registers, three waves
        // per SIMD with the smallest wave tiles, else two.  That, and the clocks of start and chunk below, are of the form of the kernel that the
        // choice was measured with; the present one starts sooner and has room for three waves with 1 x 7, 1 x 8 and 2 x 4 blocks too.
        // Other figures take other tiles, which nobody has measured against these.)
        auto estimate = [&](double N) {
            const double wgs = std::ceil(N / g.NS) * g.tiles_p * g.ndb, per_cu = std::ceil(wgs / kNumCU);
            const int room = kMaxLdsBytes / std::max(g.lds_bytes, 1);
            const double resident = std::min(per_cu, (double)std::max(1, split ? std::min(wpc, room) : std::min((g.MW < 4 && g.MW * g.NW <= 4 ? 12 : 8) / g.waves, room)));
            const double clocks = thr / 256 * resident >= 2.0 ? 22.0 : 32.0;
            const double group = split ? 4.0 : (double)(g.waves / g.KG);      // waves that share a step
            const double mfma = (double)steps * g.MW * g.NW * group / 4.0 * products * clocks;
            const double l1 = ((double)steps * group * g.MW * terms * 1024 + (double)g.npos_s * L.C * p.ex) / 64.0;
            const double lds = (double)steps * group * g.NW * terms * 1024 / 128.0 + (double)g.npos_s * L.C * p.ex / 16.0 +
                               (g.KG > 1 && !split ? 16.0 * (g.KG == 2 ? group : g.waves) * g.MW * g.NW : 0.0);
            return 8000.0 * std::ceil(per_cu / resident) + 3000.0 * g.nchunks * per_cu / resident + per_cu * std::max(mfma, std::max(l1, lds));
        };
        Choice& c = best[kg != 0];
        const double time = estimate(32.0);
        if (time < c.time) c = Choice{time, estimate(128.0), r, g};
    }
    const Choice& c = best[1].time < best[0].time && best[1].time128 <= best[0].time128 ? best[1] : best[0];
    if (!(c.time < INFINITY)) return false;
    *out = c.tuning;
    *mgeom = c.geom;
    return true;
}

// ------------------------------------------------------------------------------------------------
// Host-side validation and row unification.
// ------------------------------------------------------------------------------------------------
static sc_status_t validate_layer(const sc_layer_t* L, sc_dtype_t dt, const float* scales,
                                  const void* codebook, Plan* p)
{
    if (!L) return SC_ERR_NULL;
    if (dt != SC_F32 && dt != SC_F16 && dt != SC_I8 && dt != SC_CB4_I8 && dt != SC_CB4_F16) return SC_ERR_UNSUPPORTED;
    if (L->C <= 0 || L->D <= 0 || L->H <= 0 || L->W <= 0 || L->R <= 0 || L->S <= 0 ||
        L->stride_h <= 0 || L->stride_w <= 0 || L->pad_h < 0 || L->pad_w < 0)
        return SC_ERR_SHAPE;
    const int64_t Hp = (int64_t)L->H + 2 * (int64_t)L->pad_h, Wp = (int64_t)L->W + 2 * (int64_t)L->pad_w;
    if (Hp < L->R || Wp < L->S) return SC_ERR_SHAPE;
    const int64_t P = (Hp - L->R) / L->stride_h + 1, Q = (Wp - L->S) / L->stride_w + 1;
    const int64_t K = (int64_t)L->C * L->R * L->S;
    const int64_t X_size = (int64_t)L->C * Hp * Wp;
    const int64_t Y_size = (int64_t)L->D * P * Q;
    if (K >= (1ll << 31) || X_size >= (1ll << 31) || Y_size >= (1ll << 31)) return SC_ERR_RANGE;
    if ((dt == SC_I8 || dt == SC_CB4_I8) && !scales) return SC_ERR_UNSUPPORTED;
    if (is_codebook(dt) && !codebook) return SC_ERR_UNSUPPORTED;
    p->L = *L;
    p->dtype = dt;
    p->Hp = (int)Hp;
    p->Wp = (int)Wp;
    p->P = (int)P;
    p->Q = (int)Q;
    p->Po = (int)P;
    p->Qo = (int)Q;
    p->X_size = X_size;
    p->ex = elem_size_x(dt);
    p->ey = elem_size_y(dt);
    return SC_OK;
}

// Copy of the caller's values as raw native-width elements, unified to [D][n] with rows sorted by
// column (stable, so equal columns keep the caller's order).
struct HostTable {
    std::vector<int32_t> len;  // stored entries per row before unification
    std::vector<int32_t> col;
    std::vector<uint8_t> val;  // native element bytes: 4 / 2 / 1 / 1 (index)
};

static sc_status_t unify_rows(const Plan& p, const int32_t* rowptr, const int32_t* colidx,
                              const void* values, int n, HostTable* t)
{
    const int D = p.L.D, wsz = elem_size_w_native(p.dtype);
    const int64_t K = (int64_t)p.L.C * p.L.R * p.L.S;
    const uint8_t* v = static_cast<const uint8_t*>(values);
    t->col.assign((size_t)D * n, 0);
    t->val.assign((size_t)D * n * wsz, 0);
    t->len.assign((size_t)D, 0);
    std::vector<int32_t> order;
    for (int d = 0; d < D; ++d) {
        const int64_t beg = rowptr[d], len = (int64_t)rowptr[d + 1] - rowptr[d];
        t->len[d] = (int32_t)len;
        for (int64_t k = beg; k < beg + len; ++k) {
            if (colidx[k] < 0 || colidx[k] >= K) return SC_ERR_CSR;
            if (is_codebook(p.dtype) && v[k] > 15) return SC_ERR_CSR;
        }
        order.resize((size_t)len);
        std::iota(order.begin(), order.end(), 0);
        std::stable_sort(order.begin(), order.end(),
                         [&](int32_t a, int32_t b) { return colidx[beg + a] < colidx[beg + b]; });
        for (int j = 0; j < n; ++j) {
            const size_t o = (size_t)d * n + j;
            if (j < len) {
                t->col[o] = colidx[beg + order[j]];
                std::memcpy(&t->val[o * wsz], v + (size_t)(beg + order[j]) * wsz, wsz);
            } else {
                // filler: explicit zero "marked non-zero", at the row's last (largest) column
                t->col[o] = len > 0 ? (t->col[(size_t)d * n + len - 1] & 0x7fffffff) : 0;
                if (is_codebook(p.dtype)) t->col[o] |= (int32_t)0x80000000;  // weight must read as 0
            }
        }
    }
    return SC_OK;
}

static void free_device(Plan* p)
{
    if (p->d_col) (void)hipFree(p->d_col);
    if (p->d_theta) (void)hipFree(p->d_theta);
    if (p->d_lam) (void)hipFree(p->d_lam);
    if (p->d_lam_slab) (void)hipFree(p->d_lam_slab);
    if (p->d_lam_slab_spare) (void)hipFree(p->d_lam_slab_spare);
    if (p->d_wl32) (void)hipFree(p->d_wl32);
    if (p->d_wl32_spare) (void)hipFree(p->d_wl32_spare);
    p->d_wl32 = p->d_wl32_spare = nullptr;
    p->d_lam_slab_spare = nullptr;
    if (p->d_wlc) (void)hipFree(p->d_wlc);
    if (p->d_seg_off) (void)hipFree(p->d_seg_off);
    if (p->d_first_j) (void)hipFree(p->d_first_j);
    p->d_wlc = nullptr;
    p->d_seg_off = p->d_first_j = nullptr;
    if (p->d_scales) (void)hipFree(p->d_scales);
    if (p->d_codebook) (void)hipFree(p->d_codebook);
    if (p->d_requant) (void)hipFree(p->d_requant);
    p->d_requant = nullptr;
    if (p->d_wfrag) (void)hipFree(p->d_wfrag);
    if (p->d_len) (void)hipFree(p->d_len);
    p->d_wfrag = nullptr;
    p->d_len = nullptr;
    p->d_col = p->d_lam = p->d_lam_slab = nullptr;
    p->d_theta = nullptr;
    p->d_scales = nullptr;
    p->d_codebook = nullptr;
}

// the shapes that multiply the dense image on the matrix cores: DENSE, for SC_F32 the split form
static bool is_densified(const sc_tuning_t& t) { return t.variant == SC_VARIANT_DENSE || is_split(t); }

static sc_status_t hip_status(hipError_t e)
{
    if (e == hipSuccess) return SC_OK;
    return e == hipErrorOutOfMemory ? SC_ERR_OOM : SC_ERR_HIP;
}

// Build the tables of tuning `t` beside the ones in use and swap them in only when every step has
// succeeded: on any error the plan keeps its previous tuning, geometry and tables untouched.
static sc_status_t install_tuning(Plan* p, const sc_tuning_t& t, const SlabGeom& g, const MfmaGeom& mg, hipStream_t stream)
{
    if (is_densified(t) && !p->d_wfrag) {
        // dense weights in MFMA operand order: built on first use, the same for every tile shape
        // (fp32 plans: three bfloat16 terms per weight; such a plan never runs DENSE)
        hipError_t e;
        unsigned char* w = nullptr;
        if ((e = hipMalloc((void**)&w, is_split(t) ? split_weight_bytes(*p) : mfma_weight_bytes(*p))) != hipSuccess) return hip_status(e);
        sc_status_t st = is_split(t) ? split_densify(*p, w, stream) : mfma_densify(*p, w, stream);
        if (st == SC_OK && hipStreamSynchronize(stream) != hipSuccess) st = SC_ERR_HIP;
        if (st != SC_OK) { (void)hipFree(w); return st; }
        p->d_wfrag = w;
    }
    if (t.variant != SC_VARIANT_SLAB || is_split(t)) {
        p->tuning = t;
        p->geom = g;
        p->mg = mg;
        return SC_OK;
    }
    const size_t cnt = (size_t)p->L.D * p->n;
    hipError_t e;
    // spare copies of the two tables that are rewritten in place: allocated on first use, then the
    // roles of (table, spare) swap with every successful install
    if (cnt && !p->d_lam_slab_spare &&
        (e = hipMalloc((void**)&p->d_lam_slab_spare, cnt * 4)) != hipSuccess) return hip_status(e);
    const bool want_wl32 = t.wsrc != 0 && t.chunk_c == 0 && p->d_wl32;
    const size_t wl_bytes = ((size_t)p->L.D * p->np + 8) * 8;
    if (want_wl32 && !p->d_wl32_spare) {
        if ((e = hipMalloc((void**)&p->d_wl32_spare, wl_bytes)) != hipSuccess) return hip_status(e);
    }
    int2* wlc = nullptr;
    int32_t *seg = nullptr, *fj = nullptr;
    auto fail = [&](sc_status_t st) {
        (void)hipStreamSynchronize(stream);
        if (wlc) (void)hipFree(wlc);
        if (seg) (void)hipFree(seg);
        if (fj) (void)hipFree(fj);
        return st;
    };
    sc_status_t st = launch_stretch(*p, p->d_lam_slab_spare, g.nsh, g.nsw, p->L.stride_h, p->L.stride_w,
                                    g.chan_pitch, g.sub_pitch, g.Qs, p->ex * (g.si ? g.pack : 1), t.chunk_c, stream);
    if (st != SC_OK) return fail(st);
    if (want_wl32) {
        // (the 8 slack entries behind the table stay zero: the pass writes the rows only)
        if ((e = hipMemsetAsync(p->d_wl32_spare, 0, wl_bytes, stream)) != hipSuccess) return fail(hip_status(e));
        st = expand_weights(*p, p->d_lam_slab_spare, p->d_wl32_spare, stream);
        if (st != SC_OK) return fail(st);
    }
    std::vector<int32_t> seg_off, first_j;      // must outlive the async copies
    if (t.chunk_c > 0) {
        // segment table of the chunked form: for every (row, chunk) the entries whose input
        // channel lies in the chunk, contiguous because rows are sorted by column; segments
        // are padded with zero weights to an even length (to whole 8-entry groups for the
        // symmetric kernel).  Counted on the host, filled by a device pass.
        const int D = p->L.D, nch = g.nchunks, RS = p->L.R * p->L.S;
        const int pad = t.pipeline == 2 ? 8 : 2;     // the symmetric kernel reads whole 8-entry groups
        seg_off.assign((size_t)D * nch + 1, 0);
        first_j.assign((size_t)D * nch, 0);
        int64_t total = 0;
        for (int d = 0; d < D; ++d) {
            int j = 0;
            for (int ch = 0; ch < nch; ++ch) {
                seg_off[(size_t)d * nch + ch] = (int32_t)total;
                first_j[(size_t)d * nch + ch] = j;
                int cnt_ = 0;
                // (ragged: the fillers, which sit behind the row's own entries, are left out)
                const int jend = t.ragged ? p->h_len[d] : p->n;
                while (j < jend && ((p->h_col[(size_t)d * p->n + j] & 0x7fffffff) / RS) / g.CC == ch) { ++j; ++cnt_; }
                total += (cnt_ + pad - 1) / pad * pad;
            }
        }
        seg_off[(size_t)D * nch] = (int32_t)total;
        if (total + 16 >= (1ll << 28)) return fail(SC_ERR_RANGE);
        if ((e = hipMalloc((void**)&wlc, (size_t)(total + 16) * 8)) != hipSuccess) return fail(hip_status(e));
        if ((e = hipMalloc((void**)&seg, seg_off.size() * 4)) != hipSuccess) return fail(hip_status(e));
        if ((e = hipMalloc((void**)&fj, std::max<size_t>(first_j.size(), 1) * 4)) != hipSuccess) return fail(hip_status(e));
        if ((e = hipMemcpyAsync(seg, seg_off.data(), seg_off.size() * 4, hipMemcpyHostToDevice, stream)) != hipSuccess) return fail(hip_status(e));
        if (!first_j.empty() && (e = hipMemcpyAsync(fj, first_j.data(), first_j.size() * 4, hipMemcpyHostToDevice, stream)) != hipSuccess) return fail(hip_status(e));
        if ((e = hipMemsetAsync(wlc, 0, (size_t)(total + 16) * 8, stream)) != hipSuccess) return fail(hip_status(e));
        st = expand_weights_chunked(*p, g, p->d_lam_slab_spare, seg, fj, wlc, stream);
        if (st != SC_OK) return fail(st);
    }
    if (hipStreamSynchronize(stream) != hipSuccess) return fail(SC_ERR_HIP);
    // ---- commit: nothing below can fail
    std::swap(p->d_lam_slab, p->d_lam_slab_spare);
    if (want_wl32) std::swap(p->d_wl32, p->d_wl32_spare);
    if (t.chunk_c > 0) {
        if (p->d_wlc) (void)hipFree(p->d_wlc);
        if (p->d_seg_off) (void)hipFree(p->d_seg_off);
        if (p->d_first_j) (void)hipFree(p->d_first_j);
        p->d_wlc = wlc;
        p->d_seg_off = seg;
        p->d_first_j = fj;
    }
    p->tuning = t;
    p->geom = g;
    p->mg = mg;
    return SC_OK;
}

// Upload the unified table, run the stretch pass, install the default tuning.
static sc_status_t finish_create(Plan* p, HostTable& tab, const float* scales, const void* codebook,
                                 hipStream_t stream)
{
    const size_t cnt = (size_t)p->L.D * p->n;
    const int wsz = elem_size_w_native(p->dtype);
    p->np = (p->n + 1) / 2 * 2;
    p->h_col = std::move(tab.col);
    p->h_len = std::move(tab.len);
    // a column stored twice in one row: legal (the entries add up), but such a table has no exact
    // dense image in the weights' own width, so the DENSE variant is not offered for it
    for (int d = 0; d < p->L.D && !p->has_dup; ++d)
        for (int j = 1; j < p->h_len[d]; ++j)
            if ((p->h_col[(size_t)d * p->n + j] & 0x7fffffff) == (p->h_col[(size_t)d * p->n + j - 1] & 0x7fffffff)) { p->has_dup = true; break; }

    // three bfloat16 terms hold a weight exactly unless it is not finite or so small that the last term
    // would leave the normal range
    if (p->dtype == SC_F32) {
        const float* w = reinterpret_cast<const float*>(tab.val.data());
        float most = 0.0f;
        p->splittable = true;
        for (size_t i = 0; i < cnt && p->splittable; ++i) {
            p->splittable = w[i] == 0.0f || (std::isfinite(w[i]) && std::fabs(w[i]) >= 0x1p-100f);
            most = std::max(most, std::fabs(w[i]));
        }
        for (int len : p->h_len) p->split_full |= len > 0 && len < 16;
        // an input is held to 2^-133, the sum of a product's small terms to 2^-147: outputs from 2^28 of that
        // on are served (the error is then a sixteenth of one rounding)
        p->split_floor = (float)std::min((double)p->n * (0x1p-105 * most + 0x1p-119), 0x1p127);
    }

    // the default launch shape first: it is pure host arithmetic.  The matrix-core tile where it applies
    // (default_dense_tuning), else the slab kernel with 16 waves per workgroup and
    // weights by scalar loads where the layer allows it, otherwise whatever the heuristic resolves
    sc_tuning_t t{};
    SlabGeom g{};
    MfmaGeom mg{};
    sc_tuning_t want{};
    want.wg_threads = 1024;
    want.wsrc = is_codebook(p->dtype) ? 0 : 1;
    sc_status_t st = resolve_tuning(*p, want, &t, &g, &mg);
    if (st != SC_OK) st = resolve_tuning(*p, sc_tuning_t{}, &t, &g, &mg);
    if (st != SC_OK) return st;
    sc_tuning_t td{};
    MfmaGeom mgd{};
    const bool dense = default_dense_tuning(*p, t.variant, &td, &mgd);

    std::vector<uint8_t> packed;
    const uint8_t* theta_src = tab.val.data();
    size_t theta_bytes = cnt * wsz;
    if (is_codebook(p->dtype)) {
        // two 4-bit indices per byte, even entry in the low nibble, over the flat [D*n] table
        packed.assign((cnt + 1) / 2, 0);
        for (size_t i = 0; i < cnt; ++i) packed[i / 2] |= (uint8_t)((tab.val[i] & 15) << ((i & 1) * 4));
        theta_src = packed.data();
        theta_bytes = packed.size();
    }
    hipError_t e;
    if (cnt) {
        if ((e = hipMalloc((void**)&p->d_col, cnt * 4)) != hipSuccess) return hip_status(e);
        if ((e = hipMalloc((void**)&p->d_lam, cnt * 4)) != hipSuccess) return hip_status(e);
        if ((e = hipMalloc((void**)&p->d_lam_slab, cnt * 4)) != hipSuccess) return hip_status(e);
        if ((e = hipMalloc(&p->d_theta, theta_bytes)) != hipSuccess) return hip_status(e);
        if (!is_codebook(p->dtype)) {
            // expanded {theta32, lambda} table plus 8 zeroed entries of slack: the symmetric kernel
            // reads whole 8-entry groups and the last one of a row may reach past the row
            const size_t wl_bytes = ((size_t)p->L.D * p->np + 8) * 8;
            if ((e = hipMalloc((void**)&p->d_wl32, wl_bytes)) != hipSuccess) return hip_status(e);
            if ((e = hipMemsetAsync(p->d_wl32, 0, wl_bytes, stream)) != hipSuccess) return hip_status(e);
        }
        if ((e = hipMemcpyAsync(p->d_col, p->h_col.data(), cnt * 4, hipMemcpyHostToDevice, stream)) != hipSuccess)
            return hip_status(e);
        if ((e = hipMemcpyAsync(p->d_theta, theta_src, theta_bytes, hipMemcpyHostToDevice, stream)) != hipSuccess)
            return hip_status(e);
    }
    if ((e = hipMalloc((void**)&p->d_len, std::max<size_t>(p->h_len.size(), 1) * 4)) != hipSuccess) return hip_status(e);
    if (!p->h_len.empty() && (e = hipMemcpyAsync(p->d_len, p->h_len.data(), p->h_len.size() * 4, hipMemcpyHostToDevice, stream)) != hipSuccess)
        return hip_status(e);
    if (scales) {
        if ((e = hipMalloc((void**)&p->d_scales, (size_t)p->L.D * 4)) != hipSuccess) return hip_status(e);
        if ((e = hipMemcpyAsync(p->d_scales, scales, (size_t)p->L.D * 4, hipMemcpyHostToDevice, stream)) != hipSuccess)
            return hip_status(e);
    }
    if (is_codebook(p->dtype)) {
        const size_t cbb = (size_t)codebook_bytes(p->dtype);
        if ((e = hipMalloc((void**)&p->d_codebook, cbb)) != hipSuccess) return hip_status(e);
        if ((e = hipMemcpyAsync(p->d_codebook, codebook, cbb, hipMemcpyHostToDevice, stream)) != hipSuccess)
            return hip_status(e);
    }
    // canonical offsets into one padded sample
    st = launch_stretch(*p, p->d_lam, 1, 1, 1, 1, p->Hp * p->Wp, 0, p->Wp, 1, 0, stream);
    if (st != SC_OK) return st;
    // the host staging buffers must outlive the async copies
    if (hipStreamSynchronize(stream) != hipSuccess) return SC_ERR_HIP;
    p->path = SC_PATH_SPARSE;
    p->dispatch.choice = -1;
    if (dense) {
        st = install_tuning(p, td, SlabGeom{}, mgd, stream);
        if (st == SC_OK) p->path = SC_PATH_DENSE;
        if (st != SC_ERR_OOM) return st;
        (void)hipGetLastError();       // (no room for the dense weights: the sparse table alone)
    }
    return install_tuning(p, t, g, mg, stream);
}

}  // namespace sc

using namespace sc;

// ------------------------------------------------------------------------------------------------
// C ABI
// ------------------------------------------------------------------------------------------------
extern "C" {

sc_status_t sparse_conv_quantize_pow2(const float* x, size_t count, int32_t total_bits, float saturate_at,
                                      int8_t* codes, int32_t* frac_bits)
{
    if (!frac_bits || (count > 0 && (!x || !codes))) return SC_ERR_NULL;
    if (total_bits < 2 || total_bits > 8 || !(saturate_at > 0.0f && saturate_at <= 1.0f)) return SC_ERR_UNSUPPORTED;
    double amax = 0.0;
    for (size_t i = 0; i < count; ++i) {
        if (!std::isfinite(x[i])) return SC_ERR_RANGE;
        amax = std::max(amax, std::fabs((double)x[i]));
    }
    const double m = (double)saturate_at * amax;
    int ib = 0;
    if (m > 0.0) {
        // ceil(log2(m)) without a logarithm: m = f * 2^e with f in [0.5, 1)
        int e = 0;
        const double f = std::frexp(m, &e);
        ib = f == 0.5 ? e - 1 : e;
    } else {
        ib = 0;
    }
    const int fb = total_bits - ib - 1;
    *frac_bits = fb;
    const double lo = -std::ldexp(1.0, total_bits - 1), hi = std::ldexp(1.0, total_bits - 1) - 1.0;
    for (size_t i = 0; i < count; ++i) {
        const double v = std::min(std::max((double)x[i], -m), m);
        const double c = std::nearbyint(std::ldexp(v, fb));   // default rounding mode: ties to even
        codes[i] = (int8_t)std::min(std::max(c, lo), hi);
    }
    return SC_OK;
}

const char* sparse_conv_status_string(sc_status_t s)
{
    switch (s) {
        case SC_OK: return "ok";
        case SC_ERR_NULL: return "null pointer argument";
        case SC_ERR_SHAPE: return "invalid layer shape or batch size";
        case SC_ERR_CSR: return "malformed sparse weight table";
        case SC_ERR_UNSUPPORTED: return "unsupported dtype, missing quantisation table, or tuning that does not fit";
        case SC_ERR_RANGE: return "sample too large for 32-bit offsets";
        case SC_ERR_OOM: return "out of memory";
        case SC_ERR_WORKSPACE: return "workspace missing or too small";
        case SC_ERR_HIP: return "HIP runtime error";
    }
    return "unknown status";
}

static sc_status_t create_common(const sc_layer_t* layer, sc_dtype_t dtype, bool csr, int32_t n_ell,
                                 const int32_t* rowptr, const int32_t* colidx, const void* values,
                                 const float* scales, const void* codebook, void* stream,
                                 sparse_conv_plan_t** out)
{
    if (!out) return SC_ERR_NULL;
    *out = nullptr;
    Plan* p = new (std::nothrow) Plan();
    if (!p) return SC_ERR_OOM;
    sc_status_t st = validate_layer(layer, dtype, scales, codebook, p);
    HostTable tab;
    std::vector<int32_t> ell_rowptr;
    if (st == SC_OK) {
        const int D = layer->D;
        if (csr) {
            if (!rowptr) st = SC_ERR_NULL;
            else if (rowptr[0] != 0) st = SC_ERR_CSR;
            else {
                int nmax = 0;
                for (int d = 0; d < D && st == SC_OK; ++d) {
                    if (rowptr[d + 1] < rowptr[d]) st = SC_ERR_CSR;
                    else nmax = std::max(nmax, rowptr[d + 1] - rowptr[d]);
                }
                p->n = nmax;
                if (st == SC_OK && rowptr[D] > 0 && (!colidx || !values)) st = SC_ERR_NULL;
                if (st == SC_OK) p->true_nnz = rowptr[D];
            }
        } else {
            if (n_ell < 0) st = SC_ERR_SHAPE;
            else if ((int64_t)n_ell * D >= (1ll << 31)) st = SC_ERR_RANGE;
            else if (n_ell > 0 && (!colidx || !values)) st = SC_ERR_NULL;
            else {
                p->n = n_ell;
                p->true_nnz = (int64_t)n_ell * D;
                ell_rowptr.resize((size_t)D + 1);
                for (int d = 0; d <= D; ++d) ell_rowptr[d] = d * n_ell;
                rowptr = ell_rowptr.data();
            }
        }
    }
    if (st == SC_OK) {
        try {
            st = unify_rows(*p, rowptr, colidx, values, p->n, &tab);
        } catch (const std::bad_alloc&) {
            st = SC_ERR_OOM;
        }
    }
    if (st == SC_OK) {
        try {
            st = finish_create(p, tab, scales, codebook, (hipStream_t)stream);
        } catch (const std::bad_alloc&) {
            st = SC_ERR_OOM;
        }
    }
    if (st != SC_OK) {
        free_device(p);
        delete p;
        return st;
    }
    *out = reinterpret_cast<sparse_conv_plan_t*>(p);
    return SC_OK;
}

sc_status_t sparse_conv_plan_create_csr(const sc_layer_t* layer, sc_dtype_t dtype,
                                        const int32_t* rowptr, const int32_t* colidx,
                                        const void* values, const float* scales,
                                        const void* codebook, void* stream,
                                        sparse_conv_plan_t** out)
{
    return create_common(layer, dtype, true, 0, rowptr, colidx, values, scales, codebook, stream, out);
}

sc_status_t sparse_conv_plan_create_ell(const sc_layer_t* layer, sc_dtype_t dtype, int32_t n,
                                        const int32_t* colidx, const void* values,
                                        const float* scales, const void* codebook, void* stream,
                                        sparse_conv_plan_t** out)
{
    return create_common(layer, dtype, false, n, nullptr, colidx, values, scales, codebook, stream, out);
}

void sparse_conv_plan_destroy(sparse_conv_plan_t* plan)
{
    if (!plan) return;
    Plan* p = reinterpret_cast<Plan*>(plan);
    if (p->libconv) library_conv_destroy(p->libconv);
    free_device(p);
    delete p;
}

sc_status_t sparse_conv_plan_info(const sparse_conv_plan_t* plan, sc_plan_info_t* info)
{
    if (!plan || !info) return SC_ERR_NULL;
    const Plan* p = reinterpret_cast<const Plan*>(plan);
    std::memset(info, 0, sizeof(*info));
    info->n = p->n;
    info->P = p->P;
    info->Q = p->Q;
    info->X_size = p->X_size;
    info->true_nnz = p->true_nnz;
    info->macs_per_sample = (int64_t)p->L.D * p->P * p->Q * p->n;
    info->useful_macs_per_sample = (int64_t)p->P * p->Q * p->true_nnz;
    info->act_bytes_per_sample = (int64_t)p->L.C * p->L.H * p->L.W * p->ex + (int64_t)p->L.D * p->P * p->Q * p->ey;
    const int64_t cnt = (int64_t)p->L.D * p->n;
    int64_t wb = cnt * 4;  // offsets
    wb += is_codebook(p->dtype) ? (cnt + 1) / 2 + codebook_bytes(p->dtype) : cnt * elem_size_w_native(p->dtype);
    if (p->d_scales) wb += (int64_t)p->L.D * 4;
    info->weight_bytes = wb;
    info->tuning = p->tuning;
    info->out_P = p->Po;
    info->out_Q = p->Qo;
    info->out_elem_bytes = p->epi.requant ? 1 : p->ey;
    if (is_split(p->tuning)) {
        info->lds_bytes = p->mg.lds_bytes;
        info->grid_size = p->last_N ? split_grid_size(p->mg, p->last_N) : 0;
    } else if (p->tuning.variant == SC_VARIANT_SLAB) {
        info->lds_bytes = p->geom.lds_bytes;
        info->grid_size = p->last_N ? slab_grid_size(*p, p->geom, p->last_N) : 0;
    } else if (p->tuning.variant == SC_VARIANT_DENSE) {
        info->lds_bytes = p->mg.lds_bytes;
        info->grid_size = p->last_N ? mfma_grid_size(*p, p->mg, p->last_N) : 0;
    } else {
        info->lds_bytes = 1024 * 8;
        info->grid_size = p->last_N ? gather_grid_size(*p, p->tuning, p->last_N) : 0;
    }
    return SC_OK;
}

sc_status_t sparse_conv_plan_debug_offsets(const sparse_conv_plan_t* plan, int32_t* host_out)
{
    if (!plan || !host_out) return SC_ERR_NULL;
    const Plan* p = reinterpret_cast<const Plan*>(plan);
    const size_t cnt = (size_t)p->L.D * p->n;
    if (cnt == 0) return SC_OK;
    if (hipDeviceSynchronize() != hipSuccess) return SC_ERR_HIP;
    if (hipMemcpy(host_out, p->d_lam, cnt * 4, hipMemcpyDeviceToHost) != hipSuccess) return SC_ERR_HIP;
    for (size_t i = 0; i < cnt; ++i) host_out[i] &= 0x7fffffff;  // drop the filler flag
    return SC_OK;
}

sc_status_t sparse_conv_plan_set_tuning(sparse_conv_plan_t* plan, const sc_tuning_t* tuning, void* stream)
{
    if (!plan || !tuning) return SC_ERR_NULL;
    Plan* p = reinterpret_cast<Plan*>(plan);
    sc_tuning_t t{};
    SlabGeom g{};
    MfmaGeom mg{};
    sc_status_t st = resolve_tuning(*p, *tuning, &t, &g, &mg);
    if (st != SC_OK) return st;
    st = install_tuning(p, t, g, mg, (hipStream_t)stream);
    if (st == SC_OK) {
        p->path = is_densified(t) ? SC_PATH_DENSE : SC_PATH_SPARSE;
        p->untuned = false;
    }
    return st;
}

sc_status_t sparse_conv_plan_set_epilogue(sparse_conv_plan_t* plan, const sc_epilogue_t* ep, const float* requant_scale, void* stream)
{
    if (!plan || !ep) return SC_ERR_NULL;
    Plan* p = reinterpret_cast<Plan*>(plan);
    if ((ep->relu != 0 && ep->relu != 1) || (ep->pool != 0 && ep->pool != 2) || (ep->requant != 0 && ep->requant != 1))
        return SC_ERR_UNSUPPORTED;
    if (ep->requant && ((p->dtype != SC_I8 && p->dtype != SC_CB4_I8) || !requant_scale)) return SC_ERR_UNSUPPORTED;
    if (ep->pool && (p->P < 2 || p->Q < 2)) return SC_ERR_UNSUPPORTED;
    float* d_rq = nullptr;
    if (ep->requant) {
        hipError_t e;
        if ((e = hipMalloc((void**)&d_rq, (size_t)p->L.D * 4)) != hipSuccess) return hip_status(e);
        if (hipMemcpy(d_rq, requant_scale, (size_t)p->L.D * 4, hipMemcpyHostToDevice) != hipSuccess) { (void)hipFree(d_rq); return SC_ERR_HIP; }
    }
    const sc_epilogue_t old_epi = p->epi;
    const int old_Po = p->Po, old_Qo = p->Qo;
    float* old_rq = p->d_requant;
    p->epi = *ep;
    p->d_requant = d_rq;
    p->Po = ep->pool ? p->P / 2 : p->P;
    p->Qo = ep->pool ? p->Q / 2 : p->Q;
    // the installed launch shape may not carry an epilogue (SLAB) or not this one (DENSE with an odd
    // tile under pooling): re-resolve it, falling back to the tile that the default rule takes under this
    // epilogue if nobody has chosen a shape, and to the GATHER default
    const bool untuned = p->untuned;
    sc_status_t st = sparse_conv_plan_set_tuning(plan, &p->tuning, stream);
    sc_tuning_t td{};
    MfmaGeom mgd{};
    if (st == SC_ERR_UNSUPPORTED && untuned && default_dense_tuning(*p, SC_VARIANT_GATHER, &td, &mgd)) {
        st = sparse_conv_plan_set_tuning(plan, &td, stream);
        if (st == SC_ERR_OOM) { (void)hipGetLastError(); st = SC_ERR_UNSUPPORTED; }
    }
    if (st == SC_ERR_UNSUPPORTED) {
        sc_tuning_t g{};
        g.variant = SC_VARIANT_GATHER;
        g.split_n = 1;
        st = sparse_conv_plan_set_tuning(plan, &g, stream);
    }
    p->untuned = untuned;
    if (st != SC_OK) {
        p->epi = old_epi; p->d_requant = old_rq; p->Po = old_Po; p->Qo = old_Qo;
        if (d_rq) (void)hipFree(d_rq);
        return st;
    }
    if (old_rq) (void)hipFree(old_rq);
    if (p->libconv) { library_conv_destroy(p->libconv); p->libconv = nullptr; }
    p->dispatch.choice = -1;
    return SC_OK;
}

sc_status_t sparse_conv_plan_get_tuning(const sparse_conv_plan_t* plan, sc_tuning_t* tuning)
{
    if (!plan || !tuning) return SC_ERR_NULL;
    *tuning = reinterpret_cast<const Plan*>(plan)->tuning;
    return SC_OK;
}

sc_status_t sparse_conv_workspace_size(const sparse_conv_plan_t* plan, int32_t N, size_t* bytes)
{
    if (!plan || !bytes) return SC_ERR_NULL;
    if (N <= 0) return SC_ERR_SHAPE;
    const Plan* p = reinterpret_cast<const Plan*>(plan);
    if (p->path == SC_PATH_LIBRARY) *bytes = library_conv_workspace(p->libconv);
    else *bytes = p->tuning.variant == SC_VARIANT_GATHER ? gather_workspace_bytes(*p, N) : 0;
    return SC_OK;
}

sc_status_t sparse_conv_workspace_size_max(const sparse_conv_plan_t* plan, int32_t N, size_t* bytes)
{
    if (!plan || !bytes) return SC_ERR_NULL;
    if (N <= 0) return SC_ERR_SHAPE;
    const Plan* p = reinterpret_cast<const Plan*>(plan);
    *bytes = std::max(gather_workspace_bytes(*p, N), library_conv_workspace(p->libconv));
    return SC_OK;
}

sc_status_t sparse_conv_forward(const sparse_conv_plan_t* plan, const void* x_dev, void* y_dev,
                                int32_t N, void* workspace_dev, size_t workspace_bytes, void* stream)
{
    if (!plan || !x_dev || !y_dev) return SC_ERR_NULL;
    if (N <= 0) return SC_ERR_SHAPE;
    const Plan* p = reinterpret_cast<const Plan*>(plan);
    if (p->path == SC_PATH_LIBRARY)
        return library_conv_forward(p->libconv, x_dev, y_dev, N, workspace_dev, workspace_bytes, (hipStream_t)stream);
    if (p->tuning.variant == SC_VARIANT_SLAB) return launch_slab(*p, x_dev, y_dev, N, (hipStream_t)stream);
    if (p->tuning.variant == SC_VARIANT_DENSE) return launch_mfma(*p, x_dev, y_dev, N, (hipStream_t)stream);
    return launch_gather(*p, x_dev, y_dev, N, workspace_dev, workspace_bytes, (hipStream_t)stream);
}

// Candidate launch shapes for this layer, in a fixed order.
static void build_candidates(const Plan& p, std::vector<sc_tuning_t>* out)
{
    out->clear();
    // fillers (zero weights that unify the row lengths) are more than 5 % of the table
    const bool uneven = p.n > 0 && p.true_nnz * 100 < (int64_t)p.L.D * p.n * 95;
    std::unordered_set<std::string> seen;
    auto push = [&](sc_tuning_t t) {
        sc_tuning_t r{};
        SlabGeom g{};
        MfmaGeom mg{};
        if (resolve_tuning(p, t, &r, &g, &mg) != SC_OK) return;
        // (the tiles on the matrix cores: wg_per_cu only bounds the chunk, shapes that differ in nothing else are one)
        sc_tuning_t c = r;
        if (is_densified(r)) c.wg_per_cu = 0;
        if (!seen.emplace(reinterpret_cast<const char*>(&c), sizeof(c)).second) return;
        out->push_back(r);
    };
    for (int ns : {1, 4, 16, 64}) {
        for (int sb : {1, 2, 4, 8}) {
            sc_tuning_t t{};
            t.variant = SC_VARIANT_GATHER;
            t.sub_batch = sb;
            t.split_n = ns;
            push(t);
        }
    }
    // the densified tile on the matrix cores (16- and 8-bit activations): output-channel block x
    // tile of positions (rows of one sample, or whole planes of several) x workgroups per CU
    if (p.dtype != SC_F32 && !p.has_dup && p.n > 0) {
        // one-shot form, the contraction split otherwise than by the default (one group of four waves, two of eight):
        // the same tiles with as many groups as there are waves for, and with blocks of 16 output channels
        for (int db : {16, 32, 64, 128}) for (int wm : {1, 2, 4}) for (int wpc : {1, 2}) for (int thr : {256, 512}) for (int kg : {1, 2, 4, 8}) {
            if (db % (16 * wm) || db / (16 * wm) > 4 || (db > 32 && db >= 2 * p.L.D) || thr / 64 % (wm * kg) || kg == thr / 256 || (db == 16 && kg < 4)) continue;
            auto base = [&]() { sc_tuning_t t{}; t.variant = SC_VARIANT_DENSE; t.tile_d = db; t.waves_m = wm; t.wg_per_cu = wpc; t.wg_threads = thr; t.buffers = kg; return t; };
            for (int tp : {1, 2, 4, 7, 8, 14, 16}) {
                if (tp >= p.P) continue;
                sc_tuning_t t = base(); t.tile_p = tp; push(t);
            }
            for (int ns : {1, 2, 4, 8, 16}) { sc_tuning_t t = base(); t.tile_p = p.P; t.sub_batch = ns; push(t); }
        }
        for (int db : {32, 64, 128}) for (int wm : {1, 2, 4}) for (int wpc : {1, 2, 3}) {
            if (db % (16 * wm) || db / (16 * wm) > 4 || (db > 32 && db >= 2 * p.L.D)) continue;
            for (int thr : {256, 512}) {
                auto base = [&]() { sc_tuning_t t{}; t.variant = SC_VARIANT_DENSE; t.tile_d = db; t.waves_m = wm; t.wg_per_cu = wpc; t.wg_threads = thr; return t; };
                // (with several blocks of output channels in the layer: also 2, 4 or 8 of them per workgroup,
                // one after the other on the resident tile)
                auto pushd = [&](sc_tuning_t t) {
                    push(t);
                    if (thr == 256 && db < p.L.D)
                        for (int dl : {2, 4, 8}) { t.split_n = dl; push(t); }
                };
                pushd(base());
                for (int tp : {1, 2, 4, 7, 8, 14, 16}) {
                    if (tp >= p.P) continue;
                    sc_tuning_t t = base(); t.tile_p = tp; pushd(t);
                }
                for (int ns : {1, 2, 4, 8, 16}) {
                    sc_tuning_t t = base(); t.tile_p = p.P; t.sub_batch = ns; pushd(t);
                }
                // pointwise layers whose planes are whole 8-byte loads: the same shapes on the natural layout
                if (is_pointwise(p.L) && (p.L.H * p.L.W * p.ex) % 8 == 0) {
                    { sc_tuning_t t = base(); t.stage_rows = 1; pushd(t); }
                    for (int tp : {1, 2, 4, 7, 8, 14, 16}) {
                        if (tp >= p.P) continue;
                        sc_tuning_t t = base(); t.stage_rows = 1; t.tile_p = tp; pushd(t);
                    }
                    for (int ns : {1, 2, 4}) {
                        sc_tuning_t t = base(); t.stage_rows = 1; t.tile_p = p.P; t.sub_batch = ns; pushd(t);
                    }
                    // ... and pipelined, the chunks copied by direct-to-LDS loads
                    if (wpc <= 2) {
                        const int cb = mfma_chan_block(p.dtype);
                        for (int cc : {cb, 2 * cb, 4 * cb}) for (int np_ : {1, 2}) {
                            if (cc >= p.L.C) continue;
                            for (int tp : {1, 2, 4, 7, 8, 14, 16, 28}) {
                                sc_tuning_t t = base(); t.stage_rows = 1; t.pipeline = 1; t.producers = np_; t.chunk_c = cc;
                                t.tile_p = std::min(tp, p.P);
                                push(t);
                            }
                        }
                    }
                }
                // the pipelined form (staging waves, chunks of one or two channel blocks): filters
                // with several taps, where a chunk is multiplied for longer than it takes to stage
                if (thr == 256 && wpc <= 2 && p.L.R * p.L.S > 1) {
                    const int cb = mfma_chan_block(p.dtype);
                    for (int cc : {cb, 2 * cb}) {
                        if (cc >= p.L.C) continue;
                        for (int tp : {1, 2, 4, 7, 8, 14, 16}) {
                            sc_tuning_t t = base(); t.pipeline = 1; t.producers = 4; t.chunk_c = cc;
                            t.tile_p = std::min(tp, p.P);
                            push(t);
                        }
                        for (int ns : {2, 4}) {
                            sc_tuning_t t = base(); t.pipeline = 1; t.producers = 4; t.chunk_c = cc; t.tile_p = p.P; t.sub_batch = ns; push(t);
                        }
                    }
                }
            }
        }
    }
    // fp32 on the matrix cores: output-channel block x wave layout (a wave owns one or two blocks of 16
    // channels) x tile x chunk, one or two workgroups per CU; layers with small planes also with the
    // chunks dealt to several workgroups
    if (p.dtype == SC_F32) {
        const int layouts[][2] = {{32, 1}, {32, 2}, {64, 2}, {64, 4}, {128, 4}};
        for (int thr : {512, 256}) for (const auto& lw : layouts) for (int cc : {0, 64, 128, 256}) for (int wpc : {1, 2}) {
            if ((lw[0] > 32 && lw[0] >= 2 * p.L.D) || (cc && cc >= p.L.C)) continue;
            auto pushk = [&](int tp, int ns) {
                sc_tuning_t t{};
                t.variant = SC_VARIANT_SLAB;
                t.pipeline = 3;
                t.ragged = uneven ? 1 : 0;
                t.wg_threads = thr;
                t.tile_d = lw[0];
                t.waves_m = lw[1];
                t.chunk_c = cc;
                t.wg_per_cu = wpc;
                t.tile_p = tp;
                t.sub_batch = ns;
                push(t);
                if (p.P * p.Q <= 256 && cc) for (int ks : {2, 4}) { t.split_n = ks; push(t); }
                // pipelined: small chunks, staged one ahead by waves of their own
                if (thr == 512 && wpc == 1 && (cc != 256 || is_pointwise(p.L))) {
                    t.split_n = 0; t.producers = 4; t.chunk_c = cc ? cc : 32; push(t);
                    // Four groups of two waves split the contraction; with them also blocks of 16 channels, which make more
                    // workgroups of a single image (us with the best shape of 32 channels and more, and of 16: 3x3 128-128 at 28 x 28 7.7, 6.7; 100-90
                    // at 27 x 31 8.0, 7.1; 1-D 300-64, batch 128 10.1, 11.3).  Offered from one layout, with small tiles and chunks, to keep the
                    // search as long as it was; larger chunks would take 512-512 at 7 x 7, one image, from 12.4 to 11.6.
                    if (lw[1] <= 2) { t.buffers = 4; push(t); }
                    if (lw[0] == 32 && lw[1] == 1 && cc <= 64 && tp <= 4) { t.tile_d = 16; push(t); }
                }
            };
            for (int tp : {1, 2, 4, 7, 8, 14, 16}) if (tp < p.P) pushk(tp, 0);
            for (int ns : {1, 2, 4}) pushk(p.P, ns);
        }
    }
    const bool pw = is_pointwise(p.L);
    const bool packable = p.dtype == SC_F16 || p.dtype == SC_I8;   // tuning.pack = 1 applies
    const bool wide = p.dtype == SC_F32 || p.dtype == SC_F16;      // tuning.pack = 2 applies
    if (pw && !is_codebook(p.dtype)) {
        for (int threads : {512, 768, 1024}) {
            for (int tq : {32, 64, 96, 128, 192, 256, 384, 512}) {
              for (int wsrc : {1, 3}) for (int np_ : {1, 2, 4}) {
                sc_tuning_t t{};
                t.producers = np_;
                t.variant = SC_VARIANT_SLAB;
                t.wsrc = wsrc;
                t.pipeline = 1;
                t.wg_per_cu = 1;
                t.wg_threads = threads;
                t.tile_p = 1;
                t.tile_q = tq;
                push(t);
                if (wide && wsrc == 1 && tq >= 256) { t.pack = 2; push(t); }
              }
            }
        }
    }
    if (pw && !is_codebook(p.dtype)) {
        for (int threads : {512, 768, 1024}) {
            for (int tq : {32, 64, 96, 128, 192, 256, 384, 512}) {
                sc_tuning_t t{};
                t.variant = SC_VARIANT_SLAB;
                t.wsrc = 1;
                t.pipeline = 2;
                t.wg_per_cu = 1;
                t.wg_threads = threads;
                t.tile_p = 1;
                t.tile_q = tq;
                push(t);
            }
        }
    }
    if (pw && !is_codebook(p.dtype)) {
        for (int tq : {64, 128, 256}) for (int cc : {32, 64, 128, 256, 512}) {
            if (cc >= p.L.C) continue;
            for (int td : {0, 32, 64, 128}) {
                if (td >= p.L.D && td != 0) continue;
                sc_tuning_t t{};
                t.variant = SC_VARIANT_SLAB;
                t.wsrc = 1;
                t.pipeline = 2;
                t.wg_per_cu = 1;
                t.wg_threads = 1024;
                t.tile_p = 1;
                t.tile_q = tq;
                t.chunk_c = cc;
                t.tile_d = td;
                push(t);
                if (packable) { t.pack = 1; push(t); t.tile_q = 2 * tq; push(t); }
                if (wide && tq >= 128) { t.pack = 2; t.tile_q = 2 * tq; push(t); }
            }
        }
    }
    if (pw && !is_codebook(p.dtype)) {
        for (int np_ : {1, 2}) for (int tq : {128, 192, 256, 384, 512}) for (int cc : {16, 32, 64, 128, 256}) {
            if (cc >= p.L.C) continue;
            for (int td : {0, 64, 128}) {
                if (td >= p.L.D && td != 0) continue;
                sc_tuning_t t{};
                t.variant = SC_VARIANT_SLAB;
                t.wsrc = 1;
                t.pipeline = 1;
                t.producers = np_;
                t.wg_per_cu = 1;
                t.wg_threads = 1024;
                t.tile_p = 1;
                t.tile_q = tq;
                t.chunk_c = cc;
                t.tile_d = td;
                push(t);
                if (packable) { t.pack = 1; push(t); }
                if (wide && (tq == 256 || tq == 512)) { t.pack = 2; push(t); t.wg_threads = 768; push(t); }
            }
        }
    }
    // the same form with producers + 1 chunk buffers (a producer wave per chunk in flight), also on
    // tile widths that cut a plane into equal tiles of whole 16-byte words
    if (pw && !is_codebook(p.dtype)) {
        const int hw = p.L.H * p.L.W, words = 16 / p.ex;
        std::vector<int> tqs = {256, 384, 512};
        for (int k : {2, 3, 4, 6, 7, 8, 12, 14, 16}) {
            const int tq = round_up((hw + k - 1) / k, words);
            if (tq >= 128 && tq <= 512 && std::find(tqs.begin(), tqs.end(), tq) == tqs.end()) tqs.push_back(tq);
        }
        for (int nb : {3, 4}) for (int tq : tqs) for (int cc : {16, 32, 64}) {
            if (cc >= p.L.C) continue;
            for (int td : {0, 64, 128}) {
                if (td >= p.L.D && td != 0) continue;
                sc_tuning_t t{};
                t.variant = SC_VARIANT_SLAB;
                t.wsrc = 1;
                t.pipeline = 1;
                t.buffers = nb;
                t.producers = nb - 1;
                t.wg_per_cu = 1;
                t.wg_threads = 1024;
                t.tile_p = 1;
                t.tile_q = tq;
                t.chunk_c = cc;
                t.tile_d = td;
                push(t);
                if (packable) { t.pack = 1; push(t); }
                if (wide) { t.pack = 2; push(t); }
            }
        }
    }
    for (int wsrc : {0, 1, 2, 3}) {
        if (wsrc != 0 && is_codebook(p.dtype)) continue;
        for (int wpc : {1, 2, 3, 4}) {
            for (int threads : {256, 512, 1024}) {
                if (pw) {
                    for (int tq : {32, 64, 96, 128, 192, 256, 384, 512}) {
                        sc_tuning_t t{};
                        t.variant = SC_VARIANT_SLAB;
                        t.wsrc = wsrc;
                        t.wg_per_cu = wpc;
                        t.wg_threads = threads;
                        t.tile_p = 1;
                        t.tile_q = tq;
                        push(t);
                        if (wide && wsrc == 1 && tq >= 256) { t.pack = 2; push(t); }
                    }
                } else {
                    for (int tp : {1, 2, 3, 4, 6, 7, 8, 14, 16}) {
                        sc_tuning_t t{};
                        t.variant = SC_VARIANT_SLAB;
                        t.wsrc = wsrc;
                        t.wg_per_cu = wpc;
                        t.wg_threads = threads;
                        t.tile_p = tp;
                        t.tile_q = p.Q;
                        push(t);
                    }
                }
            }
        }
    }
    // channel-chunked one-shot form on pointwise layers: for planes too small or too oddly sized
    // for the persistent forms
    if (pw && !is_codebook(p.dtype) && p.n > 0) {
    // (deep layers with small planes: the more channels per chunk the better -- fewer, longer
    // (row, chunk) segments -- up to the whole LDS for one workgroup)
        for (int wpc : {1, 2, 3}) for (int cc : {32, 64, 128, 256, 384, 512, 768, 1024}) {
            if (cc >= p.L.C || (cc > 256 && wpc > 1)) continue;
            for (int td : {0, 32, 64, 128}) {
                if (td >= p.L.D && td != 0) continue;
                for (int tq : {64, 128, 256}) {
                    sc_tuning_t t{};
                    t.variant = SC_VARIANT_SLAB;
                    t.wsrc = 1;
                    t.wg_per_cu = wpc;
                    t.wg_threads = 1024;
                    t.tile_p = 1;
                    t.tile_q = tq;
                    t.chunk_c = cc;
                    t.tile_d = td;
                    push(t);
                    t.wsrc = 3;
                    push(t);
                }
            }
        }
    }
    // the same with several samples per workgroup, for planes of at most one wave of positions
    if (!is_codebook(p.dtype) && p.n > 0 && p.P * (p.Q + (p.L.S - 1) / p.L.stride_w) <= 64) {
        for (int wpc : {1, 2, 3}) for (int cc : {16, 32, 64, 128, 192, 256, 384, 512, 768}) {
            if (cc >= p.L.C || (cc > 256 && wpc > 1)) continue;
            for (int td : {0, 32, 64, 128}) {
                if (td >= p.L.D && td != 0) continue;
                for (int ns : {2, 4}) {
                    sc_tuning_t t{};
                    t.variant = SC_VARIANT_SLAB;
                    t.wsrc = 1;
                    t.wg_per_cu = wpc;
                    t.wg_threads = 1024;
                    t.tile_p = pw ? 1 : p.P;
                    t.tile_q = pw ? p.P * p.Q : p.Q;
                    t.chunk_c = cc;
                    t.tile_d = td;
                    t.sub_batch = ns;
                    push(t);
                    t.wsrc = 3;
                    push(t);
                }
            }
        }
    }
    // channel-chunked one-shot form (any layer shape): tiles several output rows high
    if (!pw && !is_codebook(p.dtype) && p.n > 0) {
        for (int wpc : {1, 2, 3}) for (int cc : {16, 32, 64, 128}) {
            if (cc >= p.L.C) continue;
            for (int td : {0, 64, 128}) {
                if (td >= p.L.D && td != 0) continue;
                for (int tp : {2, 4, 7, 8, 14, 16, 28}) {
                    sc_tuning_t t{};
                    t.variant = SC_VARIANT_SLAB;
                    t.wsrc = 1;
                    t.wg_per_cu = wpc;
                    t.wg_threads = 1024;
                    t.tile_p = tp;
                    t.tile_q = p.Q;
                    t.chunk_c = cc;
                    t.tile_d = td;
                    push(t);
                    t.wsrc = 3;
                    push(t);
                }
            }
        }
    }
    // 16- and 8-bit activations: the chunked one-shot form with packed positions (one LDS read per
    // 2 or 4 positions), tiles of up to 8 positions per lane
    // (interleaved samples in fp32: every shape also with the samples staged by rows)
    auto pushr = [&](sc_tuning_t t) {
        push(t);
        if (t.pack == 3 && p.dtype == SC_F32) { t.stage_rows = 1; push(t); }
    };
    if ((packable || wide) && p.n > 0) {
        for (int wpc : {1, 2, 3}) for (int cc : {16, 24, 32, 48, 64, 96, 128, 256, 384, 512}) {
            const bool odd_cc = cc == 24 || cc == 48 || cc == 96;    // with interleaved samples only
            if ((cc > p.L.C && cc != 16) || (cc > 256 && wpc > 1)) continue;
            for (int td : {0, 4, 8, 16, 32, 64, 128}) {   // (4 .. 16: with interleaved samples only -- enough workgroups on small layers)
                if (td >= p.L.D && td != 0) continue;
                for (int tile : {1, 2, 4, 7, 8, 14, 16, 28}) for (int pk : {1, 2, 3}) {
                    if ((pk == 1 && !packable) || (pk == 2 && !wide) || (pk == 3 && pw) || (tile == 1 && pk != 3) || (td != 0 && td <= 16 && pk != 3)) continue;
                    if (odd_cc && pk != 3) continue;
                    sc_tuning_t t{};
                    t.variant = SC_VARIANT_SLAB;
                    t.wsrc = 1;
                    t.wg_per_cu = wpc;
                    t.wg_threads = 1024;
                    t.tile_p = pw ? 1 : tile;
                    t.tile_q = pw ? 32 * tile : p.Q;     // pointwise: 64 .. 512 (and 224, 896 -> clipped by the fit)
                    t.chunk_c = cc;
                    t.tile_d = td;
                    t.pack = pk;
                    pushr(t);
                    // layers with fewer tiles than CUs: the chunks of a tile dealt to several workgroups
                    // (wide output-channel blocks, so that the input is staged few times)
                    if ((p.dtype == SC_F32 || p.dtype == SC_I8) && p.P * p.Q <= 256 && (td == 0 || td >= 64) && cc < p.L.C) {
                        for (int ks : {2, 4, 8}) {
                            sc_tuning_t t2 = t;
                            t2.split_n = ks;
                            pushr(t2);
                        }
                    }
                    // small planes: several sample groups along the lanes (refused unless they fit a wave)
                    if (pk == 3 && tile * (p.Q + (p.L.S - 1) / p.L.stride_w) <= 32) {
                        for (int sg : {2, 4, 8}) {
                            sc_tuning_t t2 = t;
                            t2.sub_batch = sg;
                            pushr(t2);
                            if ((p.dtype == SC_F32 || p.dtype == SC_I8) && (td == 0 || td >= 32) && cc < p.L.C)
                                for (int ks : {2, 4, 8}) { sc_tuning_t t3 = t2; t3.split_n = ks; pushr(t3); }
                            if (p.L.D >= 256) { t2.wg_threads = 256; pushr(t2); t2.wg_threads = 512; pushr(t2); }
                        }
                    }
                    // (twelve waves: two such workgroups share a CU where the registers allow, one
                    // staging while the other multiplies)
                    if (pk == 3 && p.dtype == SC_F32) { t.wg_threads = 768; pushr(t); }
                }
            }
        }
    }
    // pointwise layers with small planes: the planes of several samples end to end in one tile of
    // packed positions (up to 512 positions)
    if (pw && (packable || wide) && p.n > 0 && 2 * p.P * p.Q <= 512) {
        for (int wpc : {1, 2}) for (int cc : {64, 128, 256, 512}) {
            if (cc > p.L.C || (cc > 256 && wpc > 1)) continue;
            for (int td : {0, 32, 64, 128}) {
                if (td >= p.L.D && td != 0) continue;
                for (int fs : {2, 4}) for (int pk : {1, 2}) {
                    if ((pk == 1 && !packable) || (pk == 2 && !wide)) continue;
                    if (fs * p.P * p.Q > 512) continue;
                    sc_tuning_t t{};
                    t.variant = SC_VARIANT_SLAB;
                    t.wsrc = 1;
                    t.wg_per_cu = wpc;
                    t.wg_threads = 1024;
                    t.tile_p = 1;
                    t.tile_q = p.P * p.Q;
                    t.chunk_c = cc;
                    t.tile_d = td;
                    t.sub_batch = fs;
                    t.pack = pk;
                    push(t);
                }
            }
        }
    }
    // A table whose rows differ in length carries fillers (zero weights that unify the rows): when
    // they are more than 5 % of it, every chunked shape is also tried with the fillers left out.
    if (uneven) {
        const size_t count = out->size();
        for (size_t k = 0; k < count; ++k) {
            sc_tuning_t t = (*out)[k];
            if (t.variant != SC_VARIANT_SLAB || t.chunk_c == 0) continue;
            t.ragged = 1;
            push(t);
        }
    }
}

sc_status_t sparse_conv_plan_num_candidates(const sparse_conv_plan_t* plan, int32_t* count)
{
    if (!plan || !count) return SC_ERR_NULL;
    std::vector<sc_tuning_t> c;
    build_candidates(*reinterpret_cast<const Plan*>(plan), &c);
    *count = (int32_t)c.size();
    return SC_OK;
}

sc_status_t sparse_conv_plan_candidate(const sparse_conv_plan_t* plan, int32_t index, sc_tuning_t* tuning)
{
    if (!plan || !tuning) return SC_ERR_NULL;
    std::vector<sc_tuning_t> c;
    build_candidates(*reinterpret_cast<const Plan*>(plan), &c);
    if (index < 0 || index >= (int32_t)c.size()) return SC_ERR_SHAPE;
    *tuning = c[index];
    return SC_OK;
}

// Ring of scratch buffer pairs for the second round of the search: large enough that a pass over it
// streams from HBM (more than twice the 256 MB last-level cache), whatever the size of one pair.
static size_t autotune_ring_slots(size_t x_bytes, size_t y_bytes)
{
    const size_t target = (size_t)512 << 20;
    return std::min<size_t>(1024, target / std::max<size_t>(x_bytes + y_bytes, 1) + 2);
}

sc_status_t sparse_conv_autotune_workspace_size(const sparse_conv_plan_t* plan, int32_t N, size_t* bytes)
{
    if (!plan || !bytes) return SC_ERR_NULL;
    if (N <= 0) return SC_ERR_SHAPE;
    const Plan* p = reinterpret_cast<const Plan*>(plan);
    const size_t x_bytes = (size_t)N * p->L.C * p->L.H * p->L.W * p->ex;
    const size_t y_bytes = (size_t)N * p->L.D * p->P * p->Q * p->ey;
    // every slot may be shifted by up to 255 bytes to copy the caller's alignment
    const size_t x_slot = (x_bytes + 255 + 255) / 256 * 256, y_slot = (y_bytes + 255 + 255) / 256 * 256;
    *bytes = (gather_workspace_bytes(*p, N) + 255) / 256 * 256 + 256 + autotune_ring_slots(x_bytes, y_bytes) * (x_slot + y_slot);
    return SC_OK;
}

// The launch-shape search over the candidates whose kind is in `kinds` (bit 0: the gather kernels,
// SC_VARIANT_GATHER and SC_VARIANT_SLAB; bit 1: the densified tile, SC_VARIANT_DENSE or the split form).  Installs
// the winner; *best_ms receives its time per launch in the second (cold) round.
static sc_status_t autotune_impl(sparse_conv_plan_t* plan, const void* x_dev, void* y_dev, int32_t N, void* workspace_dev,
                                 size_t workspace_bytes, void* stream, int kinds, float* best_ms)
{
    if (!plan || !x_dev || !y_dev) return SC_ERR_NULL;
    if (N <= 0) return SC_ERR_SHAPE;
    Plan* p = reinterpret_cast<Plan*>(plan);
    hipStream_t s = (hipStream_t)stream;
    std::vector<sc_tuning_t> cands;
    build_candidates(*p, &cands);
    cands.erase(std::remove_if(cands.begin(), cands.end(), [&](const sc_tuning_t& c) {
                    return !(kinds & (is_densified(c) ? 2 : 1));
                }), cands.end());
    if (cands.empty()) return SC_ERR_UNSUPPORTED;
    const size_t gather_ws = gather_workspace_bytes(*p, N);
    if (workspace_bytes < gather_ws || (gather_ws && !workspace_dev)) return SC_ERR_WORKSPACE;
    const sc_tuning_t entry = p->tuning;          // re-installed if the search fails
    const bool had_dense = p->d_wfrag != nullptr; // (else the dense weights are given back if no shape on them wins)
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return SC_ERR_HIP;
    if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return SC_ERR_HIP; }
    sc_status_t st = SC_OK;
    // mean time of `reps` launches of the installed tuning (negative: a call failed, st says how)
    auto time_launches = [&](int reps) -> float {
        if (hipEventRecord(e0, s) != hipSuccess) { st = SC_ERR_HIP; return -1.0f; }
        for (int r = 0; r < reps && st == SC_OK; ++r)
            st = sparse_conv_forward(plan, x_dev, y_dev, N, workspace_dev, workspace_bytes, stream);
        if (st != SC_OK) return -1.0f;
        if (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess) { st = SC_ERR_HIP; return -1.0f; }
        float ms = 0;
        if (hipEventElapsedTime(&ms, e0, e1) != hipSuccess) { st = SC_ERR_HIP; return -1.0f; }
        return ms / (float)reps;
    };
    std::vector<std::pair<float, int>> timed;     // (ms per launch, candidate)
    for (size_t i = 0; i < cands.size() && st == SC_OK; ++i) {
        st = sparse_conv_plan_set_tuning(plan, &cands[i], stream);
        if (st == SC_ERR_UNSUPPORTED) { st = SC_OK; continue; }
        // (no room for the dense weights: the shapes on them are no candidates)
        if (st == SC_ERR_OOM && is_densified(cands[i]) && !p->d_wfrag) { (void)hipGetLastError(); st = SC_OK; continue; }
        if (st != SC_OK) break;
        // one warm-up launch, then enough repeats for a stable mean
        st = sparse_conv_forward(plan, x_dev, y_dev, N, workspace_dev, workspace_bytes, stream);
        // (a launch shape the caller's pointers rule out -- direct-to-LDS copies and packed stores
        // need aligned x / y -- is skipped, not an error)
        if (st == SC_ERR_UNSUPPORTED) { st = SC_OK; continue; }
        if (st != SC_OK) break;
        const float ms1 = time_launches(1);
        if (ms1 < 0) break;
        const int reps = (int)std::min(50.0f, std::max(3.0f, 2.0f / std::max(ms1, 1e-3f)));
        const float ms = time_launches(reps);
        if (ms < 0) break;
        timed.emplace_back(ms, (int)i);
    }
    // The search above runs back to back on one buffer pair, which the 256 MB last-level cache may
    // hold, while a caller that streams fresh activations pays DRAM, and the order of the candidates
    // can differ between the two.  The few fastest are therefore timed again, over a longer run
    // that rotates over a ring of scratch copies of x (and as many y buffers) larger than twice
    // that cache, each at the caller's alignment.  The ring lies in the caller's workspace behind the
    // part the launch shapes use when the workspace holds sparse_conv_autotune_workspace_size bytes,
    // else it is allocated here for the duration of the call; if neither works the round runs on
    // the caller's pair.  The best of that round is kept.
    float best = INFINITY;
    int best_i = -1;
    if (st == SC_OK && !timed.empty()) {
        std::sort(timed.begin(), timed.end());
        // finalists: the eight fastest, and the two fastest of every kernel family (variant, pipeline,
        // packing, samples per workgroup, split) not among them -- near-identical shapes of one family
        // must not crowd out the family that wins once the buffers rotate
        {
            auto family = [&](int i) {
                const sc_tuning_t& c = cands[i];
                // (shapes that deal the chunks of a tile to several workgroups, or keep a ring of chunk
                // buffers, are families of their own)
                const int split = (c.variant == SC_VARIANT_SLAB && c.split_n > 1) ? 1 : 0;
                return (c.variant << 13) | (c.stage_rows << 12) | (c.pipeline << 8) | (c.pack << 4) | (split << 3) | (c.buffers > 2 ? 4 : 0) |
                       (c.sub_batch > 1 ? 2 : 0) | (c.chunk_c > 0 ? 1 : 0);
            };
            // (two per family: the shape of a family that is fastest on cache-resident buffers is not
            // always its fastest once they rotate)
            std::vector<int> seen;
            size_t keep = std::min<size_t>(timed.size(), 8);
            for (size_t k = 0; k < keep; ++k) seen.push_back(family(timed[k].second));
            for (size_t k = keep; k < timed.size() && keep < 28; ++k) {
                const int f = family(timed[k].second);
                if (std::count(seen.begin(), seen.end(), f) >= 2) continue;
                seen.push_back(f);
                std::swap(timed[keep], timed[k]);
                ++keep;
            }
            timed.resize(keep);
        }
        const size_t finalists = timed.size();
        const size_t x_bytes = (size_t)N * p->L.C * p->L.H * p->L.W * p->ex;
        const size_t y_bytes = (size_t)N * p->L.D * p->P * p->Q * p->ey;
        const size_t x_mis = reinterpret_cast<uintptr_t>(x_dev) & 255, y_mis = reinterpret_cast<uintptr_t>(y_dev) & 255;
        const size_t x_slot = (x_bytes + x_mis + 255) / 256 * 256, y_slot = (y_bytes + y_mis + 255) / 256 * 256;
        size_t ring = autotune_ring_slots(x_bytes, y_bytes);
        unsigned char* pool = nullptr;
        bool pool_owned = false;
        {
            // the caller's workspace first: behind the part the launch shapes use, from the next
            // 256-byte boundary
            const uintptr_t w0 = reinterpret_cast<uintptr_t>(workspace_dev);
            const uintptr_t ring0 = (w0 + gather_ws + 255) / 256 * 256;
            if (workspace_dev && ring0 + ring * (x_slot + y_slot) <= w0 + workspace_bytes)
                pool = reinterpret_cast<unsigned char*>(ring0);
        }
        if (!pool) {
            size_t free_b = 0, total_b = 0;
            if (hipMemGetInfo(&free_b, &total_b) == hipSuccess)        // leave a quarter of what is free alone
                ring = std::min(ring, std::max<size_t>(2, free_b / 4 * 3 / (x_slot + y_slot)));
            if (hipMalloc((void**)&pool, ring * (x_slot + y_slot)) != hipSuccess) { pool = nullptr; (void)hipGetLastError(); }
            pool_owned = pool != nullptr;
        }
        for (size_t r = 0; pool && r < ring; ++r)
            if (hipMemcpyAsync(pool + r * x_slot + x_mis, x_dev, x_bytes, hipMemcpyDeviceToDevice, s) != hipSuccess) st = SC_ERR_HIP;
        for (size_t k = 0; k < finalists && st == SC_OK; ++k) {
            const int i = timed[k].second;
            st = sparse_conv_plan_set_tuning(plan, &cands[i], stream);
            if (st != SC_OK) break;
            st = sparse_conv_forward(plan, x_dev, y_dev, N, workspace_dev, workspace_bytes, stream);
            if (st != SC_OK) break;
            int reps = (int)std::min(200.0f, std::max(10.0f, 8.0f / std::max(timed[k].first, 1e-3f)));
            float ms;
            if (pool) {
                reps = (int)std::max<size_t>(reps, std::min<size_t>(ring, 400));   // at least once round the ring
                if (hipEventRecord(e0, s) != hipSuccess) { st = SC_ERR_HIP; break; }
                for (int r = 0; r < reps && st == SC_OK; ++r)
                    st = sparse_conv_forward(plan, pool + (r % ring) * x_slot + x_mis,
                                             pool + ring * x_slot + (r % ring) * y_slot + y_mis, N,
                                             workspace_dev, workspace_bytes, stream);
                if (st != SC_OK) break;
                if (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                    hipEventElapsedTime(&ms, e0, e1) != hipSuccess) { st = SC_ERR_HIP; break; }
                ms /= (float)reps;
            } else {
                ms = time_launches(reps);
                if (ms < 0) break;
            }
            timed[k].first = ms;
            best = std::min(best, ms);
        }
        if (pool_owned) {
            (void)hipStreamSynchronize(s);
            (void)hipFree(pool);
        }
        // Among finalists within 2 % of the fastest, take the widest tile: the longest contiguous
        // run per channel row.
        int best_tq = -1;
        for (size_t k = 0; k < finalists && st == SC_OK; ++k) {
            const sc_tuning_t& c = cands[timed[k].second];
            if (timed[k].first <= best * 1.02f && c.tile_q > best_tq) { best_tq = c.tile_q; best_i = timed[k].second; }
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (st == SC_OK && best_i < 0) st = SC_ERR_UNSUPPORTED;
    if (st == SC_OK) st = sparse_conv_plan_set_tuning(plan, &cands[best_i], stream);
    if (st != SC_OK) {
        // leave the plan as it was found
        (void)hipStreamSynchronize(s);
        (void)sparse_conv_plan_set_tuning(plan, &entry, stream);
    }
    if (!had_dense && p->d_wfrag && !is_densified(p->tuning)) {
        (void)hipStreamSynchronize(s);
        (void)hipFree(p->d_wfrag);
        p->d_wfrag = nullptr;
    }
    if (st != SC_OK) return st;
    p->last_N = N;
    if (best_ms) *best_ms = best;
    return SC_OK;
}

sc_status_t sparse_conv_plan_autotune(sparse_conv_plan_t* plan, const void* x_dev, void* y_dev,
                                      int32_t N, void* workspace_dev, size_t workspace_bytes, void* stream)
{
    return autotune_impl(plan, x_dev, y_dev, N, workspace_dev, workspace_bytes, stream, 3, nullptr);
}

// Per-layer dispatch: steps 3 and 4 of the paper's "Main scheme" (compare the layer's time in the
// sparse kernel with the dense convolution's, then configure the network layer by layer).
sc_status_t sparse_conv_plan_dispatch(sparse_conv_plan_t* plan, const void* x_dev, void* y_dev, int32_t N,
                                      void* workspace_dev, size_t workspace_bytes, void* stream, sc_dispatch_t* out)
{
    if (!plan || !x_dev || !y_dev || !out) return SC_ERR_NULL;
    if (N <= 0) return SC_ERR_SHAPE;
    Plan* p = reinterpret_cast<Plan*>(plan);
    hipStream_t s = (hipStream_t)stream;
    sc_dispatch_t r{};
    r.sparse_ms = r.dense_ms = r.library_ms = -1.0f;
    // leg 1: the gather kernels, tuned
    sc_status_t st = autotune_impl(plan, x_dev, y_dev, N, workspace_dev, workspace_bytes, stream, 1, &r.sparse_ms);
    if (st != SC_OK) return st;
    r.sparse_tuning = p->tuning;
    // leg 2: the densified tile on the matrix cores, tuned
    st = autotune_impl(plan, x_dev, y_dev, N, workspace_dev, workspace_bytes, stream, 2, &r.dense_ms);
    if (st == SC_OK) r.dense_tuning = p->tuning;
    else if (st == SC_ERR_UNSUPPORTED) r.dense_ms = -1.0f;
    else return st;
    // leg 3: the dense library on the same buffers, in the same regime as the other two: launches
    // back to back over the caller's pair after a warm-up
    if (p->libconv) { library_conv_destroy(p->libconv); p->libconv = nullptr; }
    st = has_epilogue(*p) ? SC_ERR_UNSUPPORTED : library_conv_create(*p, x_dev, y_dev, N, s, &p->libconv);
    if (st == SC_OK) {
        const size_t lws = library_conv_workspace(p->libconv);
        void* d_ws = nullptr;
        bool own_ws = false;
        if (lws <= workspace_bytes && (lws == 0 || workspace_dev)) d_ws = workspace_dev;
        else if (hipMalloc(&d_ws, lws) == hipSuccess) own_ws = true;
        else { d_ws = nullptr; (void)hipGetLastError(); }
        hipEvent_t e0, e1;
        if ((lws == 0 || d_ws) && hipEventCreate(&e0) == hipSuccess) {
            if (hipEventCreate(&e1) == hipSuccess) {
                const size_t wsz = own_ws ? lws : workspace_bytes;
                sc_status_t ls = SC_OK;
                for (int i = 0; i < 3 && ls == SC_OK; ++i) ls = library_conv_forward(p->libconv, x_dev, y_dev, N, d_ws, wsz, s);
                const int reps = 30;
                if (ls == SC_OK && hipEventRecord(e0, s) == hipSuccess) {
                    for (int i = 0; i < reps && ls == SC_OK; ++i) ls = library_conv_forward(p->libconv, x_dev, y_dev, N, d_ws, wsz, s);
                    float ms = 0;
                    if (ls == SC_OK && hipEventRecord(e1, s) == hipSuccess && hipEventSynchronize(e1) == hipSuccess &&
                        hipEventElapsedTime(&ms, e0, e1) == hipSuccess)
                        r.library_ms = ms / (float)reps;
                }
                (void)hipEventDestroy(e1);
            }
            (void)hipEventDestroy(e0);
        }
        (void)hipStreamSynchronize(s);
        if (own_ws) (void)hipFree(d_ws);
        if (r.library_ms < 0) { library_conv_destroy(p->libconv); p->libconv = nullptr; }
    } else if (st != SC_ERR_UNSUPPORTED) {
        return st;
    }
    // the library's figure is cache-warm (one buffer pair) while the other two rotate over a cold
    // ring: it is taken only when it wins by more than that difference can explain (10 %)
    r.choice = SC_PATH_SPARSE;
    float best = r.sparse_ms;
    if (r.dense_ms >= 0 && r.dense_ms < best) { best = r.dense_ms; r.choice = SC_PATH_DENSE; }
    if (r.library_ms >= 0 && r.library_ms < 0.9f * best) { best = r.library_ms; r.choice = SC_PATH_LIBRARY; }
    const sc_tuning_t& t = r.choice == SC_PATH_DENSE ? r.dense_tuning : r.sparse_tuning;
    st = sparse_conv_plan_set_tuning(plan, &t, stream);
    if (st != SC_OK) return st;
    p->path = r.choice;                 // (set_tuning selects the library's own kernels; the library path is opted into here)
    p->last_N = N;
    p->dispatch = r;
    *out = r;
    return SC_OK;
}

sc_status_t sparse_conv_plan_set_path(sparse_conv_plan_t* plan, int32_t path, void* stream)
{
    if (!plan) return SC_ERR_NULL;
    Plan* p = reinterpret_cast<Plan*>(plan);
    if (p->dispatch.choice < 0) return SC_ERR_UNSUPPORTED;          // nothing measured yet
    if (path == SC_PATH_LIBRARY) {
        if (!p->libconv) return SC_ERR_UNSUPPORTED;
        p->path = SC_PATH_LIBRARY;
        return SC_OK;
    }
    if (path != SC_PATH_SPARSE && path != SC_PATH_DENSE) return SC_ERR_UNSUPPORTED;
    if (path == SC_PATH_DENSE && p->dispatch.dense_ms < 0) return SC_ERR_UNSUPPORTED;
    return sparse_conv_plan_set_tuning(plan, path == SC_PATH_DENSE ? &p->dispatch.dense_tuning : &p->dispatch.sparse_tuning, stream);
}

}  // extern "C"
