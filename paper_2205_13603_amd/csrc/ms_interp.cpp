// Trace interpreter and validator: decisions -> kernel template parameters
// (the split / reorder / bind / cache-read / unroll / vectorize / tensorize
// schedule of Table 2, applied in a fixed order per kernel family), plus the
// hardware-limit checks of the paper's "Trace validation" paragraph.
// Host only.
#include "ms_internal.h"

#include <algorithm>
#include <cinttypes>
#include <cstdio>
#include <cstring>

using namespace ms;

namespace {

struct Reject {
    int32_t code;
};

int32_t reject(const char *fmt, ...) __attribute__((format(printf, 1, 2)));
int32_t reject(const char *fmt, ...)
{
    char buf[1024];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    return fail(MS_ERR_INVALID_TRACE, "invalid trace: %s", buf);
}

int64_t cat_value(const ms_space *sp, const ms_trace *t, int32_t slot_id, int64_t dflt)
{
    int pos;
    const ms_slot *s = find_slot(sp, slot_id, &pos);
    if (!s) return dflt;
    return s->candidates[t->d[pos].v[0]];
}

bool get_tile(const ms_space *sp, const ms_trace *t, int32_t slot_id, int32_t *f)
{
    int pos;
    const ms_slot *s = find_slot(sp, slot_id, &pos);
    if (!s) return false;
    for (int i = 0; i < 4; ++i) f[i] = (int32_t)t->d[pos].v[i];
    return true;
}

// ---------------------------------------------------------------- bodies
//
// Where no choice of factors spells out a good kernel, a rule gives the trace another body (ms_variant_params.body).  Such
// a body reads the operator and its own tile only, so every trace that a rule takes is one kernel with one key.

// Split of the whole-vector row kernel: lanes of a wavefront that share a row, vectors of each (the last one masked),
// rows and threads of a workgroup of four wavefronts.
struct RowVectors {
    int lanes, vectors, rows, threads;
};
RowVectors row_vectors_split(const ms_op *op, int v)
{
    RowVectors r = {1, 0, 0, 256};
    while (r.lanes < 64 && r.lanes * v < op->K) r.lanes *= 2;
    auto vectors = [&](int lanes) { return (int)((op->K / v + lanes - 1) / lanes); };
    // Rows of 2-byte values are bound by the exponentials, masked lanes included: narrower groups with fewer masked vectors, as long as
    // they read 128 bytes and more at a time.  206464 x 304 in fp16: 64 lanes 61 us, 16 lanes 44; 25024 x 672: 15.2, 32 lanes 12.7;
    // 200000 x 136: 32 lanes 29.8, 8 lanes 22.1.  Where fewer than four wavefronts per compute unit would be left, a launch waits for one
    // row's chain instead (1024 x 1064: 64 lanes 3.45, 32 lanes 4.0; 4096 x 304, 16 lanes: 3.45 and 3.3).
    // Not for a seventh fewer (30016 x 1320, 32 lanes: 13.8 and 13.6; 50048 x 552: 32 lanes 20.9, 16 lanes 21.3); fp32 rows are bound
    // by memory, where wide groups write whole lines (55104 x 336: 64 lanes 21.9, 32 lanes 22.9).
    if (v == 8)
        for (int lanes : {32, 16, 8}) {
            if (lanes >= r.lanes || op->M * lanes < 4 * 256 * 64 || vectors(lanes) > 8 || vectors(lanes) * v > g_limits.max_acc_per_thread) continue;
            const int now = r.lanes * vectors(r.lanes), then = lanes * vectors(lanes);
            if (lanes == 32 ? then * 6 <= now * 5 : then * 5 <= now * 4) r.lanes = lanes;
        }
    r.vectors = vectors(r.lanes);
    r.rows = r.threads / r.lanes;
    return r;
}

// Whether a nest that reads its rows once per pass (cache_read 0) is worth keeping: few long rows, each in one trip of a lane
// group of its own of at least a wavefront.  The passes then meet in the caches, and more lanes than the row kernel's 64
// share the exponentials of a row: 256 x 4096 in fp32 with 512 lanes 3.5 against 5.7 us, 64 x 2048 with 256 lanes 2.8
// against 3.5, 1024 x 4096 7.8 against 8.8.  Rows of up to 1024 elements come out even; with more rows in a launch the second
// and third pass cost bandwidth (16384 x 4096 with 256 lanes: 133 against 105).
bool keeps_wide_groups(const ms_op *op, const ms_variant_params *p)
{
    return op->K > 1024 && op->M <= 1024 && p->ti[1] == 1 && p->ti[2] <= 4 && p->ti[3] == 1 && p->tk[0] == 1 && p->tk[1] <= 16 && p->tk[2] >= 64;
}

// MS_BODY_ROW_VECTORS: elements per vector of the whole-vector row kernel (reduce.hip), 0 = not taken.
// Taken for a softmax whose lane groups read less than a 128-byte line per access, or read the row once per pass
// (cache_read 0), where a row is whole 16-byte vectors and at most 64 values per lane of a wavefront.
int row_vectors(const ms_op *op, const ms_variant_params *p)
{
    if (op->d.kind != MS_OP_SOFTMAX) return 0;
    const int v = 16 / std::max(op->in_size, op->out_size);
    if (op->K % v || op->K > 64 * 64) return 0;
    const RowVectors r = row_vectors_split(op, v);
    if (r.threads > g_limits.max_threads || r.threads / 64 > g_limits.max_waves || r.vectors * v > g_limits.max_acc_per_thread) return 0;
    if ((int64_t)p->tk[2] * p->tk[3] * op->in_size < 128) return v;
    return p->cache_read || keeps_wide_groups(op, p) ? 0 : v;
}

// Threads of the strip kernel: one per strip and channel of an image, at most 256 in a workgroup.
int64_t dw_strip_items(const ms_op *op, int64_t strip) { return ((op->OH + strip - 1) / strip) * ((op->OW + strip - 1) / strip) * op->d.dims[3]; }
int64_t dw_strip_threads(const ms_op *op, int64_t strip) { return std::min<int64_t>(256, (dw_strip_items(op, strip) + 63) / 64 * 64); }

// Whether a nest is worth keeping where strips could run: small launches (at most one strip wavefront per compute unit)
// that wait for one thread's chain of loads, not for memory.  A nest whose threads make one patch each, unrolled, straight
// from global memory, no larger than a strip's, neighbours in a row beside each other in a wavefront, is never slower there
// (137 such nests of 64 operators: 0.48 to 1.00 of the strips' time, 0.73 in the mean; 2 x 211 x 211 x 4, 5 x 5, stride 2:
// 3.1 against 6.8 us, 57 x 57 x 144, stride 2: 3.0 against 4.6).  From one wavefront per compute unit on strips win, and
// without these conditions most nests lose at every size.
bool keeps_small_launch(const ms_op *op, const ms_variant_params *p, int64_t strip)
{
    const ms_op_desc &d = op->d;
    const int64_t sp_h = (strip - 1) * d.stride + d.dims[4], sp_w = (strip - 1) * d.stride + d.dims[5];
    const int64_t ph = (int64_t)(p->ti[3] - 1) * d.stride + d.dims[4], pw = (int64_t)(p->tj[3] - 1) * d.stride + d.dims[5];
    return d.dims[0] * dw_strip_items(op, strip) <= 256 * 64 && !p->cache_read && p->unroll > 0 &&
           (int64_t)p->ti[1] * p->tj[1] * p->tc[1] * (p->tc[3] / p->vec) == 1 && ph * pw <= sp_h * sp_w &&
           (int64_t)p->tj[2] * p->tc[2] >= 32 && p->threads * 2 >= p->waves * 64;
}

// MS_BODY_STRIPS: output pixels per side of a thread's strip in the strip kernel (dwconv.hip), 0 = not taken.
// Taken where an output extent above 2 has no divisor from 3 to 8: perfect tiles then leave a thread a row, a column or a
// single pixel, which reads its inputs several times over (57 x 57 x 144, stride 2, batch 128: 75 against 50 us; 73 x 73 x 32,
// batch 22: 119 against 6).
// And taken whatever the extents in launches of more than four strip wavefronts per compute unit, from 8 output pixels a side on
// (fewer leave too much of a strip masked): strips read an input 2.25 times (3 x 3, stride 1) and keep many loads in flight,
// where nests are bound by reading it more often or by few lanes and long chains.  274 nests of 23 operators: at least 1.11 times
// the strips' time, 4.6 times in the mean (64 x 56 x 56 x 96: 35.1 against 22.0 us with 2 x 7 pixels per thread; 29 x 91 x 91 x 128
// with single pixels: 121 against 51).  Smaller launches keep their nests: there the factors can say better what fits.
int dw_strip(const ms_op *op, const ms_variant_params *p)
{
    const ms_op_desc &d = op->d;
    auto stubborn = [](int64_t e) {
        for (int64_t f = 3; f <= 8; ++f)
            if (e % f == 0) return false;
        return e > 2;
    };
    const bool many = op->OH >= 8 && op->OW >= 8 && d.dims[0] * dw_strip_items(op, 4) > 4 * 256 * 64;
    if (!stubborn(op->OH) && !stubborn(op->OW) && !many) return 0;
    const int64_t strip = 4, regs = ((strip - 1) * d.stride + d.dims[4]) * ((strip - 1) * d.stride + d.dims[5]) + d.dims[4] * d.dims[5];
    if (regs > g_limits.max_acc_per_thread || dw_strip_threads(op, strip) > g_limits.max_threads) return 0; // patch and taps stay in registers
    // 32-bit byte offsets inside an image, 32-bit counts of its strips
    if (d.dims[1] * d.dims[2] * d.dims[3] > 0x7ffffff0 / 4 || op->OH * op->OW * d.dims[3] > 0x7ffffff0) return 0;
    return keeps_small_launch(op, p, strip) ? 0 : (int)strip;
}

// The image-row kernel for first layers (conv_rows.hip): workgroups of four wavefronts of tm x tn intrinsic tiles.
struct ConvRows {
    int tm, tn, threads;
    int64_t px, tpr, tiles; // output pixels of a workgroup, workgroups of an output row (0: tiles cross rows) and plane
    int64_t lead, cpr, steps; // unused elements before a run, 8-element chunks of a run, k steps of a filter plane
    int64_t groups;      // workgroups of one instance
    int64_t lds;         // bytes of a workgroup
    int64_t regs;        // registers of a lane: accumulators, fragments, the next filter plane on its way, about 60 others
    // estimate of a launch: rounds of the workgroups that the chip holds (two per compute unit, one where the LDS is too
    // large), each a staging round trip of about three tiles' time and the tiles of a wavefront
    int64_t cost(int64_t instances) const { return (groups * instances + slots() - 1) / slots() * (3 + tm * tn); }
    int64_t slots() const { return 2 * lds > 160 * 1024 ? 256 : 512; }
};
ConvRows conv_rows_tiles(const ms_op *op, int tm)
{
    const ms_op_desc &d = op->d;
    const int64_t W = d.dims[2], Cin = d.dims[3], Cout = d.dims[4], KH = d.dims[5], KW = d.dims[6], S = d.stride, waves = 4, ohw = op->OH * op->OW;
    ConvRows c;
    c.tm = tm;
    c.tn = Cout / 32 % 2 == 0 ? 2 : Cout / 32 % 3 == 0 ? 3 : 1;
    c.threads = (int)waves * 64;
    c.px = waves * tm * 32;
    // Rows of at least two tiles: a tile keeps to its row and stages the columns it meets.  Whole rows would be read once per
    // tile and leave one workgroup per compute unit: 64 x 16384 x 4 -> 64, width 7: 73 us with whole rows, 34 so (the im2col
    // loop 40); 8 x 128 x 2048 x 4 -> 64, 3 x 3: 88 and 67; 128 x 1024 x 4 -> 32, 5 x 5: 6.7 and 5.6.  From one tile per row
    // on, the masked rest of a row costs more than it saves (8 x 128 x 640 x 4 -> 64: 23.3 and 26.2).
    c.tpr = op->OW >= 2 * c.px ? (op->OW + c.px - 1) / c.px : 0;
    c.tiles = c.tpr ? op->OH * c.tpr : (ohw + c.px - 1) / c.px;
    c.lead = d.pad * Cin % 2;
    c.cpr = (c.lead + KW * Cin + 7) / 8;
    c.steps = (KH * c.cpr + 1) / 2;
    const int64_t bn = c.tn * 32, halo = ((d.pad * Cin + c.lead) * 2 + 15) / 16 * 16;
    const int64_t last = halo - (d.pad * Cin + c.lead) * 2 + ((c.tpr ? c.px : op->OW) - 1) * S * Cin * 2 + c.cpr * 16; // end of the last run
    const int64_t row = c.tpr ? last : std::max(halo + W * Cin * 2, last);
    const int64_t rows = c.tpr ? KH : (std::min(c.px % op->OW ? (op->OW + c.px - 2) / op->OW + 1 : c.px / op->OW, op->OH) - 1) * S + KH;
    c.lds = std::max(rows * ((row + 15) / 16 * 16) + c.steps * 16 * (bn * 2 + 32), waves * 32 * (bn * op->out_size + 16));
    c.groups = c.tiles * (Cout / bn) * op->OD * d.dims[0];
    const int64_t vectors = (rows * (c.tpr ? (row + 15) / 16 : W * Cin / 8) + c.threads - 1) / c.threads + (KH * KW * Cin * bn / 8 + c.threads - 1) / c.threads;
    c.regs = tm * c.tn * 16 + (tm + c.tn) * 4 + (op->kd > 1 ? vectors * 4 : 0) + 60;
    return c;
}

bool conv_rows_fits(const ConvRows &t)
{
    return t.tm * t.tn <= 8 && t.groups <= 0x7fffffff && t.lds <= g_limits.max_lds_bytes && t.threads <= g_limits.max_threads &&
           t.threads / 64 <= g_limits.max_waves && t.tm * t.tn * 16 <= g_limits.max_acc_per_thread &&
           t.regs <= 256; // two workgroups per compute unit; 16 x 224 x 224 x 4, 7 x 7 x 7 with tm = 4 spills 56 registers: 346 us, with 2 170
}

// tm of the image-row kernel for launches over many instances, 0 = the one for one instance.  That one is chosen to spread one
// instance over the chip; where many instances fill it, larger tiles stage less per pixel.  224 x 224 x 3 -> 64, 7 x 7, stride 2
// x 256: 182, 148, 139 us with tm = 1, 2, 4 (4.2, 5.2, 7.3 for one instance); 16 x 224 x 224 x 3 -> 64, 7 x 7 x 7, stride 2 x 8:
// 156, 137, 125 (29.2, 23.7, 27.0).  Of 32 columns tm = 4 gains at most 5 % over 2 and loses up to 14 % on small images.
int conv_rows_many(const ms_op *op, int tm)
{
    int best = tm;
    auto per_pixel = [](const ConvRows &t) { return (double)(3 + t.tm * t.tn) / (double)(t.tm * t.slots()); };
    for (int t : {4, 2}) {
        const ConvRows c = conv_rows_tiles(op, t);
        if (t > tm && conv_rows_fits(c) && (c.tn > 1 || t <= 2) && per_pixel(c) < per_pixel(conv_rows_tiles(op, best))) best = t;
    }
    return best > tm ? best : 0;
}

// MS_BODY_IMAGE_ROWS: tm of the image-row kernel, 0 = not taken.  Taken for 1 to 4 channels per pixel where the cache-read
// of X is not shared by several tiles (compute_at 0, 1), where the im2col loader and the patch of single elements read
// 2-byte elements (3-D: 573 -> 127 us for 8 x 16 x 224 x 224 x 3 -> 64, 7 x 7 x 7, stride 2, and 9.6 -> 7.7 us for one
// 8 x 64 x 64 x 1, 5 x 5 x 5; 2-D in filter rows: 117 -> 72.5 us for 128 x 224 x 224 x 3 -> 64, 7 x 7, and 7.8 us on both
// sides, which is a launch, for one 64 x 64 x 3).
int conv_rows(const ms_op *op, const ms_variant_params *p)
{
    const ms_op_desc &d = op->d;
    if (d.kind != MS_OP_CONV2D_NHWC || p->family != MS_FAM_GEMM_MFMA || p->compute_at > 1 || p->rfactor > 1) return 0;
    const int64_t H = d.dims[1], W = d.dims[2], Cin = d.dims[3], Cout = d.dims[4], S = d.stride;
    if (op->nb != 1 || d.dilation != 1 || Cin > 4 || (d.in_dtype != MS_F16 && d.in_dtype != MS_BF16)) return 0;
    // whole 16-byte vectors per image row, runs at even elements, whole intrinsic columns
    if (W * Cin % 8 || S * Cin % 2 || Cout % 32) return 0;
    if (op->depth * H * W * Cin > 0x7fffffff / 2 || op->OH * op->OW > 0x7fffffff / 2) return 0;
    int best = 0;
    double cost = 0;
    for (int tm : {4, 2, 1}) {
        const ConvRows t = conv_rows_tiles(op, tm);
        if (!conv_rows_fits(t)) continue;
        const double c = (double)((t.groups + 511) / 512) * (3 + tm * t.tn);
        if (!best || c < cost) {
            best = tm;
            cost = c;
        }
    }
    return best;
}

// MS_BODY_PHASES: output phases (stride^2) of a transposed convolution whose rows can be ordered by phase, 0 = not taken.
// Taken where every tile keeps to one phase and every k step to one tap: the k loop then covers that phase's taps only.
// Elsewhere (filters that the stride does not divide, tiles wider than a phase) all taps are walked.
int conv_phases(const ms_op *op, const ms_variant_params *p)
{
    const ms_op_desc &d = op->d;
    const int64_t S = d.stride;
    if (d.kind != MS_OP_CONV2D_TRANSPOSED_NHWC || p->family != MS_FAM_GEMM_MFMA || S < 2 || op->nb != 1 || p->cache_read > 4) return 0;
    if (d.dims[5] % S || d.dims[6] % S || op->OH % S || op->OW % S) return 0;
    if ((d.dims[0] * (op->OH / S) * (op->OW / S)) % p->block_m || d.dims[3] % p->block_k || op->K % p->block_k) return 0;
    return p->tk[0] % (S * S * std::max(1, p->rfactor)) ? 0 : (int)(S * S);
}

// MS_BODY_DOUBLE_STEPS: LDS stages of 128-byte rows in the double-step form of the ping-pong ring (gemm_mfma.hip, PP_STAGES),
// 0 = not taken.  Taken for every ring of 64- or 128-byte k tiles under the ping-pong order (cache_read 8, 9, 10) whose reduction is
// whole 128-byte rows: a load of a k-contiguous operand then covers whole cache lines (46.6 bytes per clock and compute unit
// from the L2 to LDS, 34 to 39 with rows of 64 bytes), and a stage is refilled part by part, up to four times as early.
// 1024 x 1024 x 1024 fp16 x 64: 154 -> 130 us, 4096^3 bf16: 123 -> 97.
// The intrinsic is the 16-row one of the same wave tile: a launch that keeps the matrix cores busy is held by the power it
// draws, and the 16-row forms run it at 1.84 GHz where the 32-row forms run at 1.62 (bf16 4096^3: 97.5 and 104 us).
// As many stages as the LDS takes, up to eight: small tiles multiply a step in one phase (rows of one slot) and need three, and
// a step of theirs takes less than a round trip to memory.
// Wave tiles that fill the register file spill here, as they do in the nest; of 22 such tiles timed on both, 20 are faster here (256 x 256
// of 4 x 8 tiles per wavefront, fp16 1024^3 x 64: 142 us, 150 in the nest; four wavefronts of 9 x 6: 145 and 229), two of int8 slower
// (ten wavefronts of 3 x 5: 230 and 206; 10 x 3: 219 and 214).
int64_t double_step_rows(const ms_variant_params *p) { return (int64_t)p->ti[1] * p->ti[3] * (p->tile_unit[0] / 16); } // 16-row tiles of a wavefront
int64_t double_step_staging(const ms_op *op, const ms_variant_params *p) // bytes of the staged output rows of all wavefronts
{
    return p->cache_write ? (int64_t)p->waves * 16 * p->tj[3] * p->tile_unit[1] * op->out_size : 0;
}
int double_steps(const ms_op *op, const ms_variant_params *p)
{
    const ms_op_desc &d = op->d;
    const int es = op->in_size;
    if (p->family != MS_FAM_GEMM_MFMA || is_conv2d(d.kind) || p->cache_read < 8 || p->reorder != 3) return 0;
    const int64_t k_row = 128 / es;                                // k elements of a 128-byte row
    if (p->block_k * (int64_t)es > 128 || op->K % k_row) return 0;
    // 32-bit byte offsets inside a workgroup's rows
    const int64_t b_span = d.b_strides[2] == 1 ? k_row * d.b_strides[1] : (int64_t)p->block_n * d.b_strides[2];
    if (std::max((int64_t)p->block_m * d.a_strides[1], b_span) > 0x7ffffff0 / es) return 0;
    const int64_t stage = (int64_t)(p->block_m + p->block_n) * 128;
    const int64_t stages = std::min<int64_t>(8, (g_limits.max_lds_bytes - double_step_staging(op, p)) / stage);
    return stages < 2 || (stages == 2 && double_step_rows(p) < 2) ? 0 : (int)stages;
}

// MS_BODY_CONV_STEPS: convolutions as matrix products on double steps (gemm_mfma.hip, CONV_STEPS).  Taken for 2-byte inputs whose
// pixels are whole 16-byte groups of channels, where the cache-read of X sits under the k0 loop (compute_at 0): that nest stages
// its im2col tile through registers with index arithmetic per load, its tiles have to divide the pixels, and a step of a
// transposed convolution may mix phases.  48 x 48 x 32 -> 128, 3 x 3, batch 256: 101 -> 67 us; 16 x 16 x 256 -> 256, dilation 2, batch 88:
// 51 -> 32; transposed 12 x 12 x 512 -> 64, 4 x 4, stride 2, batch 72: 123 -> 28; 16 x 16 x 256 -> 128, batch 64: 27.4 -> 22.2.
struct ConvSteps {
    int bm, bn, wi, wj, stages;      // workgroup tile, wavefronts, LDS stages of 128-byte rows
    int64_t phases, th, tw;          // output phases (stride^2 of a transposed convolution), taps of one
    int64_t tiles, steps;            // tiles and 128-byte k steps of one phase
    int64_t lds, cost;
};
ConvSteps conv_steps_tile(const ms_op *op, int bm, int bn)
{
    const ms_op_desc &d = op->d;
    ConvSteps c;
    c.bm = bm;
    c.bn = bn;
    c.wj = bn == 32 ? 1 : bn == 256 || (bn == 128 && bm < 256) ? 4 : 2;
    c.wi = 8 / c.wj;
    const int64_t S = d.kind == MS_OP_CONV2D_TRANSPOSED_NHWC ? d.stride : 1;
    c.phases = S * S;
    c.th = d.dims[5] / S;
    c.tw = d.dims[6] / S;
    const int64_t rows = d.dims[0] * (op->OH / S) * (op->OW / S), staging = 8 * 16 * (bn / c.wj) * op->out_size, stage = (bm + bn) * 128;
    c.tiles = (rows + bm - 1) / bm;
    c.steps = (c.th * c.tw * d.dims[3] + 63) / 64;
    c.stages = (int)std::min<int64_t>(8, (g_limits.max_lds_bytes - staging) / stage);
    c.lds = c.stages * stage + staging;
    // clocks of a launch: rounds of 256 workgroups; a step is bound by the matrix cores or by its bytes from the L2, a tile starts and
    // ends with nothing beside it.  One image is launched over many instances (16 here) or is bound by the launch itself.
    const int64_t launch = c.tiles * c.phases * (op->N / bn) * (d.dims[0] == 1 ? 16 : 1);
    c.cost = (launch + 255) / 256 * (2500 + c.steps * std::max<int64_t>(bm * bn / 24, (bm + bn) * 3) + bm * bn / 16);
    return c;
}
// tile of the body as bm * 1000 + bn, 0 = not taken
int conv_steps(const ms_op *op, const ms_variant_params *p)
{
    const ms_op_desc &d = op->d;
    if (!is_conv2d(d.kind) || p->family != MS_FAM_GEMM_MFMA || op->nb != 1 || is_3d(op) || op->in_size != 2 || p->compute_at || p->cache_read > 4 ||
        p->rfactor > 1 || p->tap_rows)
        return 0;
    const bool transposed = d.kind == MS_OP_CONV2D_TRANSPOSED_NHWC;
    const int64_t S = transposed ? d.stride : 1, Cin = d.dims[3];
    if (Cin < 32 || Cin % (transposed ? 64 : 8) || op->N % (transposed ? 64 : 32)) return 0;
    // nests of small tiles (pixels with few divisors) lose to it everywhere
    const bool small_nest = p->block_m * p->block_n < 64 * 32;
    // single images of few channels: the search has better locations for X (56 x 56 x 64 -> 64, 3 x 3, x 512: 143 us resident)
    if (d.dims[0] == 1 && Cin <= 64 && op->N <= 64 && !small_nest) return 0;
    // one k step per tile leaves nothing to overlap (20 x 20 x 64, 1 x 1, x 512: 20.2 and 20.4 us), and steps of several taps cost index
    // arithmetic that narrow tiles do not hide (14 x 14 x 32 -> 64, 3 x 3, batch 512: 12.7 and 13.4; -> 256: 32.3 and 28.3)
    // (transposed 8 x 8 x 128 -> 64, 2 x 2, batch 256, two steps: 6.05 and 6.24; 24 x 24 x 64 -> 256, batch 96, one step: 42.4 and 26.9;
    // half a step, 16 x 16 x 32 -> 128, 1 x 1, batch 512: 9.4 and 10.1; 28 x 28 x 32 -> 256, batch 256: 32.9 and 23.3)
    const int k_of_tap_set = op->K / (S * S);
    if (op->N <= 64 && k_of_tap_set <= (transposed ? 128 : 64)) return 0;
    if (op->N <= 128 && k_of_tap_set < 64) return 0;
    if (Cin % 64 && op->N < 128 && !small_nest) return 0;
    // short reductions into 32 columns (14 x 14 x 256 -> 32, 1 x 1, batch 200: 6.5 and 7.3), and small batches of the several-tap kind
    // (8 x 14 x 14 x 96 -> 32, 3 x 3: 7.7 and 9.7)
    if ((op->N == 32 && op->K < 512) || (Cin % 64 && op->N < 128 && d.dims[0] > 1 && op->M < 4096)) return 0;
    if (d.dims[5] % S || d.dims[6] % S || op->OH % S || op->OW % S || d.dims[5] / S > 15 || d.dims[6] / S > 15) return 0;
    // 32-bit byte offsets from the image stack and inside the k-rows of a step.  The kernel's offsets start ahead of the stack, by
    // the padding or by the taps of a phase (PIX_0, TAP_0 in gemm_mfma.hip), and end before the buffer does (0x7ffffff0)
    const int64_t ahead = (transposed ? (d.dims[5] / S - 1) * d.dims[2] + d.dims[6] / S - 1 : op->pad_h * d.dims[2] + d.pad) * Cin * 2;
    if (d.dims[0] * d.dims[1] * d.dims[2] * Cin * 2 + ahead > 0x7ffffff0 || (op->K + 64) * op->N > 0x3fffffff) return 0;
    if (op->M > 0x7fffffff - 256) return 0; // 32-bit numbers of pixels, those of the last tile that are masked among them
    if (g_limits.max_threads < 512 || g_limits.max_waves < 8) return 0;
    int best = 0;
    int64_t cost = 0;
    for (int bn : {256, 128, 96, 64, 32})
        for (int bm : {256, 128, 64}) {
            if (op->N % bn || (bn == 32 && bm < 128) || bm * bn > 256 * 128) continue; // 256 x 256 spills
            const ConvSteps c = conv_steps_tile(op, bm, bn);
            if (c.stages < 2 || bm * bn / 512 > g_limits.max_acc_per_thread || c.tiles * c.phases * (op->N / bn) > 0x7fffffff) continue;
            if (c.stages < 3 && bm / c.wi < 32) continue; // one slot per step needs three stages
            if (!best || c.cost < cost) {
                best = bm * 1000 + bn;
                cost = c.cost;
            }
        }
    return best;
}

// MS_BODY_FEW_ROWS: products of few rows with a row-major matrix (gemm_rows.hip), the second kernel of a nest's variant
// (fill_kernel, takes_fill).
struct FewRows {
    int mt, nc;                 // 16-row tiles and 16-column tiles of a workgroup
    int waves, depth, lds;      // wavefronts that share its reduction, their blocks of 64 k values in flight
    int64_t tiles;
};
FewRows few_rows_tile(const ms_op *op, int tile)
{
    FewRows c;
    c.mt = tile & 15;
    c.nc = tile >> 4 & 15;
    c.waves = tile >> 8 & 31;
    c.depth = tile >> 16;
    c.tiles = op->M / (c.mt * 16) * (op->N / (c.nc * 16));
    int g = c.mt;
    while (c.mt % g || (g > 1 && c.waves * g * c.nc * 1024 > 64 * 1024)) --g;
    c.lds = c.waves * std::max(g * c.nc * 1024, c.mt * 2048);
    return c;
}
// its tile, 0 = not taken
int few_rows(const ms_op *op)
{
    const ms_op_desc &d = op->d;
    if (d.kind != MS_OP_GEMM || op->in_size != 2 || op->M > 128 || op->M % 16 || op->N % 32 || op->K % 64) return 0;
    // rows of B that lanes read side by side, 16-byte groups of k values of A, 32-bit offsets of elements
    if (d.a_strides[2] != 1 || d.b_strides[2] != 1 || d.a_strides[1] % 8 || d.b_strides[1] % 8) return 0;
    if (op->K * d.b_strides[1] > 0x7fffffff || op->M * d.a_strides[1] > 0x7fffffff) return 0;
    // below 1 MiB of weights launches take the 3.5 us that any launch takes
    if (op->K * op->N < 512 * 1024) return 0;
    int best = 0;
    int64_t cost = 0;
    for (int nc : {2, 4})
        for (int mt = 1; mt <= 8; ++mt) {
            if (op->M / 16 % mt || op->N % (nc * 16)) continue;
            // eight wavefronts hide latency better than four (48 x 4096 x 2048, mt = 1: 6.9 us and 7.3) until their sums are many
            // (48 x 8000 x 1536, mt = 3: 7.5 and 7.2)
            const int tile = mt | nc << 4 | (mt <= 2 ? 8 : 4) << 8 | (mt <= 2 ? 2 : 3) << 16;
            const FewRows c = few_rows_tile(op, tile);
            if (c.lds > g_limits.max_lds_bytes || c.waves > g_limits.max_waves || c.waves * 64 > g_limits.max_threads) continue;
            if (mt * nc * 4 > g_limits.max_acc_per_thread || c.tiles > 1024) continue;
            // a k value costs lookups of mt + 4 groups of four lanes (columns by 32: of mt + 2, at half the bytes for a line of the L2,
            // which comes to the same); a second round overlaps the first in part (112 x 2176 x 1280, mt = 1: 238 tiles of 64 columns
            // 5.3 us, 476 of 32 6.2)
            const int64_t rounds = (c.tiles + 255) / 256, clocks = op->K * (mt + 4) * (rounds == 1 ? 5 : rounds * 4);
            if (!best || clocks < cost) {
                best = tile;
                cost = clocks;
            }
        }
    return best;
}

// MS_BODY_CONV_PLANES: first layers on persistent workgroups over filter planes (conv_planes.hip), the second kernel of a variant on
// MS_BODY_IMAGE_ROWS (fill_kernel, takes_fill).
struct ConvPlanes {
    int tm, tn;
    int64_t steps;                   // k steps of a filter plane
    int64_t tiles, lds, clocks;      // tiles of an instance, bytes of a workgroup, estimate for a tile
    int waves() const { return 4; }
    int per_cu() const { return 2 * lds <= 160 * 1024 ? 2 : 1; }
};
ConvPlanes conv_planes_tile(const ms_op *op, int tm)
{
    const ms_op_desc &d = op->d;
    const int64_t W = d.dims[2], Cin = d.dims[3], Cout = d.dims[4], KH = d.dims[5], KW = d.dims[6], S = d.stride, ohw = op->OH * op->OW;
    ConvPlanes c;
    c.tm = tm;
    c.tn = Cout / 32 % 2 == 0 ? 2 : 1;
    const int64_t px = c.waves() * tm * 32, lead = d.pad * Cin % 2, cpr = (lead + KW * Cin + 7) / 8, steps = c.steps = (KH * cpr + 1) / 2, bn = c.tn * 32;
    const int64_t halo = ((d.pad * Cin + lead) * 2 + 15) / 16 * 16, last = halo - (d.pad * Cin + lead) * 2 + (op->OW - 1) * S * Cin * 2 + cpr * 16;
    const int64_t units = (std::max(halo + W * Cin * 2, last) + 15) / 16;
    const int64_t rows = (std::min(px % op->OW ? (op->OW + px - 2) / op->OW + 1 : px / op->OW, op->OH) - 1) * S + KH;
    const int64_t stage = ((rows * units + 63) / 64 + (steps * 16 * bn / 8 + 63) / 64) * 1024;
    c.lds = stage + (d.has_bias ? 2048 : 0);
    c.tiles = (ohw + px - 1) / px * (Cout / bn) * op->OD * d.dims[0];
    // a plane: products of the two wavefronts of a SIMD, their LDS reads at 128 bytes per clock; what a load's latency leaves; results
    const int64_t n = c.per_cu();
    c.clocks = op->kd * (std::max(n * steps * tm * c.tn * 32, n * steps * (tm + c.tn) * 32) + 1500) + n * tm * c.tn * 500;
    return c;
}
int conv_planes(const ms_op *op)
{
    const ms_op_desc &d = op->d;
    // columns of 96 channels would leave as parts of lines (128 x 128 x 3 -> 96, 3 x 3, batch 115: 20.4 us and 26.2)
    if (op->out_size != 2 || op->in_size != 2 || op->N / 32 % 3 == 0) return 0;
    if (d.dims[1] * d.dims[2] * d.dims[3] > 0x0fffffff || op->K * op->N > 0x3fffffff) return 0; // 32-bit byte offsets, ahead of a plane and behind it too
    // planes of few steps hide no loads (3-D, 192 x 192 x 3 -> 32, 3 x 3 x 3, x 11: 15.2 us on image rows and 17.0)
    if (op->kd > 1 && conv_planes_tile(op, 1).steps < 4) return 0;
    int best = 0;
    double cost = 0;
    for (int tm : {4, 3, 2, 1}) {
        const ConvPlanes c = conv_planes_tile(op, tm);
        if (tm * c.tn > 8 || c.lds > g_limits.max_lds_bytes || c.tiles > 0x7fffffff || c.waves() > g_limits.max_waves || c.waves() * 64 > g_limits.max_threads) continue;
        if (tm * c.tn * 16 > g_limits.max_acc_per_thread) continue;
        const int64_t slots = 256 * c.per_cu();
        const double clocks = d.dims[0] == 1 ? (double)c.tiles / slots * c.clocks : (double)((c.tiles + slots - 1) / slots) * c.clocks;
        if (!best || clocks < cost) {
            best = tm;
            cost = clocks;
        }
    }
    return best;
}

// MS_BODY_CONV_PATCH: convolutions of stride 1 from input patches in LDS (conv_patch.hip), the second kernel of a convolution's
// variant (fill_kernel, takes_fill).  Not for filters of one column, which read every input once, nor for strides: of nine layers
// at stride 2 four were slower than their nests and gathers (48 x 48 x 64 -> 64, batch 512: 46.6 us and 52.9; 20 x 20 x 256 -> 256, batch
// 176: 34.5 and 44.9), and transposed ones by phases share too few taps (16 x 16 x 256 -> 128, 4 x 4, batch 64: 22.0 and 27.3).
constexpr int CONV_PATCH_MANY = 1 << 25; // in a tile's code: chosen for launches over many instances too
struct ConvPatch {
    int cw, r, tn;                   // a wavefront's tile: a strip of cw columns (of 16 / cw bands of rows), rows, 16-channel tiles
    int ws, wr, wj;                  // wavefronts over strips, rows and channels
    bool whole;                      // a tile is whole images
    int rows, imgs;                  // rows of an image, images of a tile
    int64_t tiles;                   // of one instance
    int64_t patch, weights, lds;     // bytes of a patch, of a step's weights, of a workgroup
    int loads;                       // load instructions of a patch and of a step's weights
    int waves, per_cu;               // that multiply, of a workgroup; workgroups on a compute unit
    int64_t clocks;                  // estimate for a tile
    int code() const { return cw | r << 5 | tn << 13 | wr << 16 | wj << 20 | whole << 24; }
};
ConvPatch conv_patch_tile(const ms_op *op, int code)
{
    const ms_op_desc &d = op->d;
    ConvPatch c;
    c.cw = code & 31;
    c.r = code >> 5 & 31;
    c.tn = code >> 13 & 7;
    c.wr = code >> 16 & 15;
    c.wj = code >> 20 & 7;
    c.whole = code >> 24 & 1;
    const int64_t dil = std::max(1, (int)d.dilation), th = d.dims[5], tw = d.dims[6], oh = op->OH, ow = op->OW;
    const int bands = 16 / c.cw;
    c.rows = c.whole ? (int)oh : bands * c.wr * c.r;
    c.imgs = c.whole ? bands * c.wr : 1;
    c.ws = (int)((ow + c.cw - 1) / c.cw);
    c.waves = c.ws * c.wr * c.wj;
    const int64_t bn = c.wj * c.tn * 16, pw = ow + (tw - 1) * dil, slots = c.imgs * (c.rows + (th - 1) * dil) * (c.cw == 4 ? pw | 1 : pw);
    c.patch = (slots + 15) / 16 * 1024;
    c.weights = th * 32 * bn * 2;
    c.loads = (int)((c.patch + c.weights) / 1024);
    c.lds = 2 * c.patch + 3 * c.weights + (d.has_bias ? 2048 : 0) + 128;
    c.per_cu = 2 * c.lds <= 160 * 1024 && c.waves <= 5 ? 2 : 1;
    c.tiles = (c.whole ? (d.dims[0] + c.imgs - 1) / c.imgs : d.dims[0] * ((oh + c.rows - 1) / c.rows)) * (op->N / bn);
    // a step: products of the wavefronts of a SIMD, their LDS reads at 128 bytes per clock, loads into LDS at 36
    const int64_t per_simd = (c.waves * c.per_cu + 3) / 4, rows_read = c.r + (th - 1) * dil;
    const int64_t chunks = d.dims[3] / 32, mfma = th * c.r * c.tn * 16, step = per_simd * mfma * 11 / 8 + 400;
    const int64_t lds = (rows_read + th * c.tn) * 8 * c.waves * c.per_cu, fill = (c.patch / tw + c.weights) / 34 * c.per_cu;
    c.clocks = chunks * tw * std::max({step, lds, fill, (int64_t)1200}) * (c.per_cu == 2 ? 27 : 20) / 20 + per_simd * c.r * c.tn * 88 + 500;
    return c;
}
int conv_patch(const ms_op *op)
{
    const ms_op_desc &d = op->d;
    if (!is_conv2d(d.kind) || op->nb != 1 || is_3d(op) || op->in_size != 2 || op->out_size != 2 || d.dims[3] % 32) return 0;
    if (d.stride > 1 || d.dims[6] < 2 || d.dims[6] > 15 || d.dims[5] > 15) return 0;
    // 32-bit byte offsets inside a filter; images of a tile, with what lies ahead of and behind them, below half of that
    if (op->K * op->N > 0x3fffffff) return 0;
    const int64_t oh = op->OH, images = std::max(d.dims[1] * d.dims[2] * d.dims[3], oh * op->OW * op->N) * 2;
    const int64_t ahead = (d.dims[5] * std::max(1, (int)d.dilation) + oh) * d.dims[2] * d.dims[3] * 2;
    int best = 0, best_many = 0; // for one instance, for many
    double cost = 0, cost_many = 0;
    for (int tn : {4, 2})
        for (int wj = 1; wj <= 4; ++wj) {
            if (op->N % (wj * tn * 16) || (tn == 2 && op->N % 64 == 0 && wj % 2)) continue; // 32 channels of a line of 64: both halves here
            for (int cw : {16, 8, 4})
                for (int64_t r = 1; r <= std::min<int64_t>(16, oh); ++r)
                    for (int wr = 1; wr <= 8; ++wr)
                        for (int whole = 0; whole <= (r == oh); ++whole) {
                            const int bands = 16 / cw;
                            if (whole ? bands * wr > d.dims[0] : (bands * wr - 1) * r >= oh) continue; // wavefronts with nothing to do
                            ConvPatch t{};
                            t.cw = cw;
                            t.r = (int)r;
                            t.tn = tn;
                            t.wr = wr;
                            t.wj = wj;
                            t.whole = whole;
                            const ConvPatch c = conv_patch_tile(op, t.code());
                            const int per_simd = (c.per_cu * (c.waves + 1) + 3) / 4;
                            if (c.waves > 15 || c.waves < 2 || c.waves >= g_limits.max_waves || (c.waves + 1) * 64 > g_limits.max_threads) continue;
                            // Registers: an address for each load, in the loads' wavefront; sums, a step's weights and at least 60 others in
                            // those that multiply
                            const int64_t budget = 512 / per_simd / 8 * 8, live = r * tn * 4 + d.dims[5] * tn * 4;
                            if (c.lds > g_limits.max_lds_bytes || c.loads > std::min<int64_t>(150, budget - 40)) continue;
                            if (live + 60 > budget || r * tn * 4 > g_limits.max_acc_per_thread) continue;
                            // 64 channels of a wavefront take half as many again for fragments and results on their way: 254 of 256 registers for
                            // 8 rows under 3 x 3, 276 where that is dilated, 266 for 7 rows under 5 x 5.  Their spills cost more than smaller
                            // tiles (56 x 56 x 64 -> 64, dilation 2, x 176: 57 us and 43; 28 x 28 x 64 -> 64, 5 x 5, x 248: 39.9 and 36.0), but in
                            // dilated layers of a batch (16 x 16 x 64 -> 128, batch 512: 22.0 and 24.7; 32 x 32 x 128 -> 256, batch 64: 32.9
                            // and 35.3).  Two registers too many at 32 channels cost nothing (40 x 40 x 64 -> 128 x 168: 44.1 and 47.3).
                            const bool dilated = d.dilation > 1;
                            if (tn == 4 && live * 3 / 2 + (dilated ? 8 : -8) > budget && !(dilated && d.dims[0] > 1)) continue;
                            if (c.imgs * images + ahead > 0x3fffffff || c.tiles > 0x7fffffff) continue;
                            const int64_t slots = 256 * c.per_cu;
                            const double clocks = (double)((c.tiles + slots - 1) / slots) * c.clocks, many = (double)c.tiles / slots * c.clocks;
                            if (!best || clocks < cost) {
                                best = c.code();
                                cost = clocks;
                            }
                            if (!best_many || many < cost_many) {
                                best_many = c.code();
                                cost_many = many;
                            }
                        }
        }
    if (!best) return 0; // no tile fits: channels that are no whole columns of 32, rows wider than 15 wavefronts
    // single images come in many instances; a batch as one
    return d.dims[0] == 1 || best == best_many ? best_many | CONV_PATCH_MANY : best;
}

void set4(int32_t *f, int64_t f0, int64_t f1, int64_t f2, int64_t f3)
{
    f[0] = (int32_t)f0;
    f[1] = (int32_t)f1;
    f[2] = (int32_t)f2;
    f[3] = (int32_t)f3;
}

// Chooses the body and, for another one than the nest, makes the launch fields of *p those of that kernel.
void resolve_body(const ms_op *op, ms_variant_params *p)
{
    const ms_op_desc &d = op->d;
    p->body = MS_BODY_NEST;
    if ((p->body_tile = row_vectors(op, p))) {
        const RowVectors r = row_vectors_split(op, p->body_tile);
        p->body = MS_BODY_ROW_VECTORS;
        p->grid[0] = (int32_t)((op->M + r.rows - 1) / r.rows);
        set4(p->ti, p->grid[0], 1, r.rows, 1);
        set4(p->tk, 1, r.vectors, r.lanes, p->body_tile);
        p->block_m = r.rows;
        p->vec = p->body_tile;
        p->unroll_k1 = r.vectors;
        p->threads = r.threads;
        p->acc_per_thread = r.vectors * p->body_tile;
        p->lds_bytes = 0;
    } else if (p->family == MS_FAM_DWCONV && (p->body_tile = dw_strip(op, p))) {
        const int64_t strip = p->body_tile;
        p->body = MS_BODY_STRIPS;
        p->threads = (int32_t)dw_strip_threads(op, strip);
        p->grid[0] = (int32_t)((dw_strip_items(op, strip) + p->threads - 1) / p->threads);
        set4(p->ti, (op->OH + strip - 1) / strip, 1, 1, strip);
        set4(p->tj, (op->OW + strip - 1) / strip, 1, 1, strip);
        set4(p->tc, d.dims[3], 1, 1, 1);
        p->block_m = p->block_n = (int32_t)strip;
        p->block_k = p->threads;
        p->vec = 1;
        p->unroll_k1 = p->unroll_k2 = 0;
        p->acc_per_thread = (int32_t)(strip * strip);
        p->lds_bytes = 0;
    } else if ((p->body_tile = conv_rows(op, p))) {
        const ConvRows c = conv_rows_tiles(op, p->body_tile);
        p->body = MS_BODY_IMAGE_ROWS;
        p->body_tile_many = conv_rows_many(op, p->body_tile);
        p->grid[0] = (int32_t)c.groups;
        p->grid[1] = p->grid[2] = 1;
        p->block_m = (int32_t)c.px;
        p->block_n = c.tn * 32;
        p->block_k = (int32_t)c.steps * 16;
        p->vec = p->vec_b = 8;
        p->threads = c.threads;
        p->acc_per_thread = c.tm * c.tn * 16;
        p->lds_bytes = (int32_t)c.lds;
    } else if ((p->body_tile = conv_steps(op, p))) {
        const ConvSteps c = conv_steps_tile(op, p->body_tile / 1000, p->body_tile % 1000);
        p->body = MS_BODY_CONV_STEPS;
        set4(p->ti, c.tiles * c.phases, 1, c.wi, c.bm / 16 / c.wi);
        set4(p->tj, op->N / c.bn, 1, c.wj, c.bn / 16 / c.wj);
        set4(p->tk, 2 * c.steps, 1, 1, 1);
        p->tile_unit[0] = p->tile_unit[1] = 16;
        p->tile_unit[2] = 32;
        p->mfma = MS_MFMA_CODE(16, 16, 32);
        p->block_m = c.bm;
        p->block_n = c.bn;
        p->block_k = 32;
        p->grid[0] = p->ti[0] * p->tj[0];
        p->grid[1] = p->grid[2] = 1;
        p->threads = 512;
        p->acc_per_thread = c.bm * c.bn / 512;
        p->lds_bytes = (int32_t)c.lds;
        p->cache_read = 10;
        p->cache_write = 1;
        p->reorder = 3;
        p->vec = p->vec_b = 8;
        p->lds_pad = p->unroll = 0;
        p->unroll_k1 = p->unroll_k2 = 1;
    } else if ((p->body_tile = double_steps(op, p))) {
        const int es = op->in_size, unit_k = 64 / es;
        p->body = MS_BODY_DOUBLE_STEPS;
        p->lds_bytes = (int32_t)(p->body_tile * (int64_t)(p->block_m + p->block_n) * 128 + double_step_staging(op, p));
        // the same wave tile in 16-row intrinsics, one of them per 64 bytes of k
        p->ti[3] *= p->tile_unit[0] / 16;
        p->tj[3] *= p->tile_unit[1] / 16;
        p->tile_unit[0] = p->tile_unit[1] = 16;
        p->tile_unit[2] = unit_k;
        p->mfma = MS_MFMA_CODE(16, 16, unit_k);
        set4(p->tk, op->K / unit_k, 1, 1, 1);
        p->block_k = unit_k;
        p->cache_read = 10; // the three rings are one kernel, its stages are body_tile
        p->vec = p->vec_b = 16 / es;
        p->unroll = 0;
        p->unroll_k1 = p->unroll_k2 = 1;
    } else {
        if ((p->body_tile = conv_phases(op, p))) p->body = MS_BODY_PHASES; // the launch is the nest's
        return;
    }
    p->waves = p->threads / 64;
}

uint64_t hash_params(const ms_op *op, const ms_variant_params *p)
{
    uint64_t h = 0x243F6A8885A308D3ull;
    auto add = [&](uint64_t v) { h = mix64(h ^ mix64(v)); };
    const ms_op_desc &d = op->d;
    add((uint64_t)d.kind);
    add((uint64_t)d.in_dtype);
    add((uint64_t)d.out_dtype);
    add((uint64_t)d.stride);
    add((uint64_t)d.pad);
    if (op->pad_h != d.pad && (is_conv2d(d.kind))) add(0x1D00000000ull + (uint64_t)op->pad_h); // 1-D convolutions only
    if (is_3d(op)) {
        add(0x3D00000000ull + (uint64_t)op->depth);
        add((uint64_t)op->kd);
    }
    add((uint64_t)d.dilation);
    add((uint64_t)d.has_bias);
    add((uint64_t)d.relu);
    for (int i = 0; i < 8; ++i) add((uint64_t)d.dims[i]);
    for (int i = 0; i < 3; ++i) {
        add((uint64_t)d.a_strides[i]);
        add((uint64_t)d.b_strides[i]);
    }
    add((uint64_t)p->family);
    if (!follows_decisions(p)) { // the operator and the body's own tile are all that such a kernel reads
        add(0xB0D7000000ull + (uint64_t)p->body);
        add((uint64_t)p->body_tile);
        if (p->body_tile_many) add((uint64_t)p->body_tile_many);
        return h;
    }
    add((uint64_t)p->mfma);
    for (int i = 0; i < 4; ++i) {
        add((uint64_t)p->ti[i]);
        add((uint64_t)p->tj[i]);
        add((uint64_t)p->tc[i]);
        add((uint64_t)p->tk[i]);
    }
    add((uint64_t)p->cache_read);
    add((uint64_t)p->vec);
    add((uint64_t)p->vec_b);
    add((uint64_t)p->cache_write);
    add((uint64_t)p->unroll_k1); // the unroll budget itself is not part of the key: the two factors it
    add((uint64_t)p->unroll_k2); // resolves to select the code, and budgets that resolve alike give one kernel
    add((uint64_t)p->lds_pad);
    add((uint64_t)p->reorder);
    add((uint64_t)p->compute_at);
    if (p->tap_rows) add(0x7A9ull);
    if (p->rfactor > 1) add(0x4F0000ull + (uint64_t)p->rfactor);
    if (p->body == MS_BODY_DOUBLE_STEPS) add(0xD0B1E0000ull + (uint64_t)p->body_tile);
    return h;
}

void unroll_factors(ms_variant_params *p)
{
    // budget = number of innermost iterations that may be unrolled; k3 is always unrolled
    int32_t u = p->unroll;
    int32_t k1 = p->tk[1], k2 = p->tk[2], k3 = p->tk[3];
    if (u <= 0) {
        p->unroll_k1 = 1;
        p->unroll_k2 = 1;
        return;
    }
    p->unroll_k2 = std::min(k2, std::max(1, u / k3));
    if (p->unroll_k2 == k2 && (int64_t)k2 * k3 <= u)
        p->unroll_k1 = std::min(k1, std::max(1, u / (k2 * k3)));
    else
        p->unroll_k1 = 1;
    // keep the unrolled body within the instruction cache: at most 4096
    // multiply-accumulate (or matrix-core) instructions per lane
    int64_t per_iter = (int64_t)std::max(1, p->acc_per_thread) * k3;
    if (p->mfma) per_iter = (int64_t)p->ti[1] * p->ti[3] * p->tj[1] * p->tj[3] * k3 * 16;
    while (p->unroll_k1 > 1 && per_iter * p->unroll_k2 * p->unroll_k1 > 4096) p->unroll_k1 = (p->unroll_k1 + 1) / 2;
    while (p->unroll_k2 > 1 && per_iter * p->unroll_k2 > 4096) p->unroll_k2 = (p->unroll_k2 + 1) / 2;
}

} // namespace

static thread_local bool t_nests_only = false; // validate_as_nest

extern "C" int32_t ms_trace_validate(const ms_op *op, const ms_space *space, const ms_trace *trace, ms_variant_params *out)
{
    if (!op || !space || !trace) return fail(MS_ERR_BAD_ARG, "ms_trace_validate: NULL argument");
    if (space->n_slots < 1 || space->n_slots > MS_MAX_SLOTS) return fail(MS_ERR_BAD_ARG, "ms_trace_validate: bad space");
    if (trace->n != space->n_slots)
        return reject("trace has %d decisions, the space has %d sampling instructions (truncated?)", trace->n, space->n_slots);
    // well-formedness of every decision, read or not
    for (int i = 0; i < space->n_slots; ++i) {
        const ms_slot &s = space->slots[i];
        const ms_decision &d = trace->d[i];
        if (d.slot_id != s.slot_id) return reject("decision %d is for slot id %d, expected %d (%s)", i, d.slot_id, s.slot_id, s.name);
        if (d.kind != s.kind) return reject("decision %d (%s) has the wrong kind", i, s.name);
        if (s.kind == MS_SLOT_CATEGORICAL) {
            if (d.n != 1) return reject("categorical %s carries %d values", s.name, d.n);
            if (d.v[0] < 0 || d.v[0] >= s.n_candidates)
                return reject("categorical %s: index %" PRId64 " outside [0,%d)", s.name, d.v[0], s.n_candidates);
            if (s.weight[d.v[0]] <= 0) return reject("categorical %s: candidate %" PRId64 " has zero probability", s.name, d.v[0]);
        } else {
            if (d.n != s.n_factors) return reject("tile %s carries %d factors, expected %d", s.name, d.n, s.n_factors);
            int64_t e = slot_extent(space, trace, i);
            if (e < 1) return reject("tile %s: extent undefined", s.name);
            int64_t prod = 1;
            for (int f = 0; f < d.n; ++f) {
                if (d.v[f] < 1) return reject("tile %s: factor %d is %" PRId64, s.name, f, d.v[f]);
                if (d.v[f] > e) return reject("tile %s: factor %d = %" PRId64 " exceeds the extent %" PRId64, s.name, f, d.v[f], e);
                prod *= d.v[f];
                if (prod > e) break;
            }
            if (prod != e) return reject("tile %s: factors multiply to %" PRId64 ", loop extent is %" PRId64, s.name, prod, e);
        }
    }

    ms_variant_params p;
    memset(&p, 0, sizeof p);
    p.family = space->family;
    const ms_op_desc &d = op->d;
    const ms_limits &L = g_limits;
    p.unroll = (int32_t)cat_value(space, trace, MS_SLOT_UNROLL, 0);
    p.vec = (int32_t)cat_value(space, trace, MS_SLOT_VECTORIZE, 1);
    p.vec_b = (int32_t)cat_value(space, trace, MS_SLOT_VECTORIZE_B, 1);
    p.cache_write = (int32_t)cat_value(space, trace, MS_SLOT_CACHE_WRITE, 0);
    p.lds_pad = (int32_t)cat_value(space, trace, MS_SLOT_STORAGE_ALIGN, 0);
    p.tap_rows = (space->flags & MS_SPACE_TAP_ROWS) && d.kind == MS_OP_CONV2D_NHWC && op->nb == 1 && !is_3d(op) && d.dilation == 1 ? 1 : 0;
    p.reorder = (int32_t)cat_value(space, trace, MS_SLOT_REORDER, 0);
    p.compute_at = (int32_t)cat_value(space, trace, MS_SLOT_COMPUTE_AT, 0);
    p.rfactor = (int32_t)cat_value(space, trace, MS_SLOT_RFACTOR, 1);

    if (space->family == MS_FAM_GEMM_ALU || space->family == MS_FAM_GEMM_MFMA) {
        if (!get_tile(space, trace, MS_SLOT_TILE_I, p.ti) || !get_tile(space, trace, MS_SLOT_TILE_J, p.tj) ||
            !get_tile(space, trace, MS_SLOT_TILE_K, p.tk))
            return fail(MS_ERR_BAD_ARG, "ms_trace_validate: the space lacks a tile slot");
        p.cache_read = (int32_t)cat_value(space, trace, MS_SLOT_CACHE_READ, 1);
        int es = op->in_size;
        if (space->family == MS_FAM_GEMM_ALU) {
            p.mfma = MS_MFMA_NONE;
            p.tile_unit[0] = p.tile_unit[1] = p.tile_unit[2] = 1;
        } else {
            p.mfma = (int32_t)cat_value(space, trace, MS_SLOT_TENSORIZE, 0);
            mfma_dims(p.mfma, &p.tile_unit[0], &p.tile_unit[1], &p.tile_unit[2]);
            if (p.tile_unit[0] != p.tile_unit[1] || (p.tile_unit[0] != 16 && p.tile_unit[0] != 32))
                return reject("tensorize: unknown intrinsic %d", p.mfma);
        }
        int64_t bm = (int64_t)p.ti[1] * p.ti[2] * p.ti[3] * p.tile_unit[0];
        int64_t bn = (int64_t)p.tj[1] * p.tj[2] * p.tj[3] * p.tile_unit[1];
        int64_t bk = (int64_t)p.tk[1] * p.tk[2] * p.tk[3] * p.tile_unit[2];
        if (bm > 4096 || bn > 4096 || bk > 4096) return reject("workgroup tile %" PRId64 "x%" PRId64 "x%" PRId64 " is beyond any register/LDS budget", bm, bn, bk);
        p.block_m = (int32_t)bm;
        p.block_n = (int32_t)bn;
        p.block_k = (int32_t)bk;
        int64_t g = (int64_t)p.ti[0] * p.tj[0];
        if (g > 0x7fffffff / std::max<int64_t>(1, op->nb)) return reject("grid of %" PRId64 " workgroups overflows", g);
        p.grid[0] = (int32_t)g;
        p.grid[1] = 1;
        p.grid[2] = (int32_t)op->nb;
        int64_t units = (int64_t)p.ti[2] * p.tj[2];
        int64_t acc;
        if (p.mfma) {
            // conv2d with helper wavefronts (compute_at 3): four more, one per SIMD, that only move data
            if (p.compute_at == 3) units += 4;
            if (units > L.max_waves) return reject("%" PRId64 " wavefronts per workgroup, the limit is %d", units, L.max_waves);
            p.waves = (int32_t)units;
            p.threads = p.waves * L.wave_size;
            acc = (int64_t)p.ti[1] * p.ti[3] * p.tj[1] * p.tj[3] * (p.tile_unit[0] * p.tile_unit[1] / L.wave_size);
        } else {
            if (units > L.max_threads) return reject("%" PRId64 " threads per workgroup, the limit is %d", units, L.max_threads);
            p.threads = (int32_t)units;
            p.waves = (p.threads + L.wave_size - 1) / L.wave_size;
            acc = (int64_t)p.ti[1] * p.ti[3] * p.tj[1] * p.tj[3];
        }
        if (p.threads > L.max_threads) return reject("%d threads per workgroup, the limit is %d", p.threads, L.max_threads);
        if (acc > L.max_acc_per_thread) return reject("%" PRId64 " accumulators per lane, the register budget is %d", acc, L.max_acc_per_thread);
        p.acc_per_thread = (int32_t)acc;
        unroll_factors(&p);
        // cache-read: LDS footprint
        int64_t lds = 0;
        if (p.mfma) {
            int kp = p.tile_unit[2] / (L.wave_size / p.tile_unit[0]); // k elements one lane feeds per intrinsic
            int64_t padb = p.lds_pad ? 16 : 0;
            // fragments of more than 16 bytes lie in LDS as 16-byte halves, each in a (padded) plane of its own
            const int split = kp * es > 16 ? kp * es / 16 : 1;
            int64_t rowsA = split * (bm * (kp / split) * es + padb), rowsB = split * (bn * (kp / split) * es + padb);
            lds = (int64_t)(p.cache_read >= 2 ? 2 : 1) * (bk / kp) * (rowsA + rowsB);
            if (p.lds_pad == 3 || p.lds_pad == 4) {
                // B row-major in LDS (dense k-rows of bn elements, granules swizzled), fragments through the transposing loads
                if (is_conv2d(d.kind) || !(d.b_strides[2] == 1 && d.b_strides[1] != 1)) return reject("storage_align 3, 4 (row-major B in LDS) is for GEMMs whose B is contiguous along j");
                if (!((es == 2 && (kp == 4 || kp == 8)) || (es == 1 && (kp == 8 || kp == 16 || kp == 32))))
                    return reject("storage_align 3, 4 needs fragments of whole transposing loads: 4 or 8 k per lane of 2-byte, 8, 16 or 32 k per lane of 1-byte inputs");
                if (p.cache_read < 1 || p.cache_read > 4) return reject("storage_align 3, 4 applies to register staging (cache_read 1..4)");
                if (p.vec_b * es != 16) return reject("storage_align 3, 4 moves B in 16-byte vectors: vectorize_b must be %d", 16 / es);
                if (d.b_strides[1] % (16 / es) || d.b_strides[0] % (16 / es)) return reject("storage_align 3, 4 needs 16-byte aligned rows of B");
                // 4: rows of B padded by 32 bytes instead of swizzled
                lds = (int64_t)(p.cache_read >= 2 ? 2 : 1) * ((bk / kp) * rowsA + bk * (bn * es + (p.lds_pad == 4 ? 32 : 0)));
            }
            if (p.cache_read >= 5) {
                // direct-to-LDS ring: dense tiles, no padding (the swizzle replaces it)
                const int ce = 16 / es; // elements per 16-byte chunk
                if (!((es == 2 && kp == 8) || (es == 1 && kp == 16)))
                    return reject("direct-to-LDS staging needs 16-byte fragments: 2-byte inputs with 8 k per lane or 1-byte inputs with 16 k per lane");
                if (bk * es != 64 && bk * es != 128 && bk * es != 256) return reject("direct-to-LDS staging needs a k tile of 64, 128 or 256 bytes, not %" PRId64, bk * es);
                if (d.a_strides[2] != 1 || d.a_strides[1] % ce || d.a_strides[0] % ce) return reject("direct-to-LDS staging needs 16-byte aligned rows of A");
                if (d.b_strides[1] == 1 && d.b_strides[2] != 1) {
                    if (d.b_strides[2] % ce || d.b_strides[0] % ce) return reject("direct-to-LDS staging needs 16-byte aligned rows of B");
                } else if (d.b_strides[2] == 1) {
                    if (d.b_strides[1] % ce || d.b_strides[0] % ce) return reject("direct-to-LDS staging needs 16-byte aligned rows of B");
                    if (bn % 16) return reject("direct-to-LDS staging reads B in groups of 16 columns");
                } else {
                    return reject("direct-to-LDS staging needs B contiguous along k or j");
                }
                if (p.lds_pad) return reject("direct-to-LDS staging has its own swizzle: storage_align must be 0");
                // the j-contiguous B tile is rounded up to whole 1 KiB load instructions
                int64_t btile = d.b_strides[2] == 1 ? ((bk * (bn / ce) + 63) / 64) * 1024 : bn * bk * es;
                const int stages = p.cache_read >= 8 ? p.cache_read - 6 : p.cache_read - 3;
                lds = (int64_t)stages * (bm * bk * es + btile);
                if (p.cache_read >= 8) {
                    // ping-pong on the ring: two groups of wavefronts one phase apart under persistent workgroups
                    if (p.reorder != 3) return reject("ping-pong on the ring (cache_read 8, 9, 10) runs under persistent workgroups: reorder must be 3");
                    if (p.waves % 2) return reject("ping-pong on the ring needs an even number of wavefronts, not %d", p.waves);
                    if (p.tk[1] != 1) return reject("ping-pong on the ring: a k0 step is k2 slots of k3 intrinsic steps, k1 must be 1");
                    // a slot's fragments and the accumulators are all live; 64 more registers hold the LDS addresses of the
                    // fragments, the load offsets and the epilogue's temporaries (what the compiler needed for a
                    // 128 x 64 wave tile: 247 registers with 128 accumulators and 48 fragment registers)
                    const int64_t fr = kp * es / 4 > 0 ? kp * es / 4 : 1;
                    const int64_t fragr = ((int64_t)p.ti[1] * p.ti[3] + (int64_t)p.tj[1] * p.tj[3]) * p.tk[3] * fr;
                    const int64_t have = 512 / ((p.waves + 3) / 4);
                    if (fragr + acc + 64 > have)
                        return reject("ping-pong on the ring: %" PRId64 " fragment + %" PRId64 " accumulator + 64 other registers per lane exceed the %" PRId64
                                      " a wavefront can have", fragr, acc, have);
                    // the k2 slots are always unrolled, whatever the budget: one kernel, one key
                    p.unroll_k1 = 1;
                    p.unroll_k2 = p.tk[2];
                }
            }
            if (is_conv2d(d.kind) && op->K % p.tile_unit[2] && !p.tap_rows) {
                // the k split covers the reduction rounded up to the intrinsic's k; only the im2col loader pads with zeros
                if (p.compute_at) return reject("KH*KW*Cin = %" PRId64 " is not a multiple of the intrinsic's k = %d: compute_at must be 0", op->K, p.tile_unit[2]);
                if (p.cache_read >= 5) return reject("a padded reduction cannot be staged directly to LDS");
            }
            if (is_3d(op) && p.compute_at) return reject("3-D convolution: compute_at must be 0 (the resident patch is a set of image rows)");
            if (p.tap_rows) {
                // the reduction as KH runs of KW * Cin contiguous elements, each rounded up to the intrinsic's k
                if (p.cache_read >= 5) return reject("filter-row layout: no direct-to-LDS staging");
                if (p.compute_at >= 1 && (d.stride * d.dims[3] * es) % 4) return reject("filter-row layout with a resident patch: pixels of an output row must start at multiples of 4 bytes");
            }
            if (p.compute_at) {
                // conv2d with the activations' cache-read under the workgroup tile loop: the input rows of
                // the tile (zero halo included) are resident, only the weights are staged per k step
                if (!is_conv2d(d.kind)) return reject("compute_location applies to conv2d only");
                if (p.compute_at == 1 && p.cache_read > 3) return reject("with the input patch resident only the weights are staged per k step: cache_read 1, 2 or 3");
                if (p.compute_at == 2 && p.cache_read > 2) return reject("with resident weights cache_read is 1 (patch loaded between tiles) or 2 (next patch prefetched)");
                if (p.compute_at == 3 && (p.cache_read != 2 || !p.cache_write))
                    return reject("helper wavefronts prefetch the patch and write the staged tile: cache_read 2 and cache_write 1");
                if (p.compute_at >= 2 && p.reorder != 0) return reject("persistent workgroups with resident weights walk the tile list in order: reorder must be 0");
                int64_t cin = d.dims[3] / op->nb, ohw = op->OH * op->OW; // channels of one group
                if (cin % p.tile_unit[2] && !p.tap_rows) return reject("resident input patch: Cin = %" PRId64 " is not a multiple of the intrinsic's k = %d", cin, p.tile_unit[2]);
                if (ohw % bm) return reject("resident input patch: the %" PRId64 "-pixel tile straddles images of %" PRId64 " output pixels", bm, ohw);
                int64_t rows = bm % op->OW == 0 ? bm / op->OW : (op->OW + bm - 2) / op->OW + 1;
                int64_t pr = (rows - 1) * d.stride + d.dilation * (d.dims[5] - 1) + 1, pw = (op->OW - 1) * d.stride + d.dilation * (d.dims[6] - 1) + 1;
                int64_t ps = cin * es + (p.lds_pad ? 16 : 0);
                if (p.tap_rows) {
                    // dense pixels (a run crosses pixel boundaries), and the pixels that the padding of the last run reads
                    const int64_t run = d.dims[6] * cin, kr = (run + p.tile_unit[2] - 1) / p.tile_unit[2] * p.tile_unit[2];
                    ps = cin * es;
                    pw += (kr - run + cin - 1) / cin;
                    if ((pw * ps) % 4) pw += 1; // rows start at multiples of 4 bytes (2-byte elements, odd Cin)
                }
                int64_t patch = pr * pw * ps;
                lds = (int64_t)(p.cache_read >= 2 ? 2 : 1) * (bk / kp) * rowsB + patch;
                if (p.compute_at >= 2) lds = (int64_t)p.tk[0] * (bk / kp) * rowsB + patch; // all k steps of the weights
                if (p.compute_at == 4) {
                    // weights in registers: LDS holds one k step of them as a staging buffer
                    lds = (bk / kp) * rowsB + patch;
                    if (p.cache_read > 2) return reject("with the weights in registers cache_read is 1 (patch loaded between tiles) or 2 (next patch prefetched)");
                }
                if ((cin * es) % 16 && p.lds_pad && !p.tap_rows) return reject("resident input patch: padded pixels need Cin * element size to be a multiple of 16 bytes");
                if (d.dims[0] * d.dims[1] * d.dims[2] * d.dims[3] > 0x7fffffff / es) return reject("resident input patch: one instance of X exceeds 32-bit byte offsets");
            }
            if (p.reorder == 3 && p.cache_read < 5) return reject("persistent workgroups (reorder 3) are built on direct-to-LDS staging (cache_read 5, 6, 7)");
            if (p.rfactor > 1) {
                // the reduction of one output tile shared by rfactor workgroups: whole runs of k0 steps each
                if (p.tk[0] % p.rfactor) return reject("rfactor %d does not divide the %d steps of the k0 loop", p.rfactor, p.tk[0]);
                if (p.reorder == 3 || p.compute_at >= 2) return reject("persistent workgroups own the whole reduction of their tiles: rfactor must be 1");
                if (p.cache_write) return reject("rfactor writes partial sums straight from the accumulators: cache_write must be 0");
                if (g * p.rfactor > 0x7fffffff / std::max<int64_t>(1, op->nb)) return reject("grid of %" PRId64 " workgroups overflows", g * p.rfactor);
                p.grid[0] = (int32_t)(g * p.rfactor);
            }
            if (p.cache_write) {
                // the output tile reuses the operand buffers: rows of bn outputs padded by 16 bytes
                int64_t ctile = bm * (bn * op->out_size + 16);
                if (p.cache_read >= 8) {
                    // one staging area per wavefront: the rows of one intrinsic tile across the wavefront's j3 adjacent tiles
                    const int64_t wrow = (int64_t)p.tj[3] * p.tile_unit[1] * op->out_size;
                    if (wrow % 16) return reject("cache_write on the ring: a wavefront's staged rows of %" PRId64 " bytes are not whole 16-byte chunks", wrow);
                    lds += (int64_t)p.waves * p.tile_unit[0] * wrow;
                } else if (p.reorder == 3 || p.compute_at >= 2) lds += ctile; // persistent workgroups keep their operands alive during the epilogue
                else if (ctile > lds) lds = ctile;
                if ((op->N * op->out_size) % 16) return reject("cache_write needs output rows that are multiples of 16 bytes");
            }
            // fragment operands of one k step for the whole wave tile live in registers too
            int64_t frag = ((int64_t)p.ti[1] * p.ti[3] + (int64_t)p.tj[1] * p.tj[3]) * p.tk[3] * (kp * es / 4 > 0 ? kp * es / 4 : 1);
            // registers that carry a tile from global memory to LDS; with two buffers they are live across the k step
            int64_t stage = (bm * bk * es / 4 + p.threads - 1) / p.threads + (bn * bk * es / 4 + p.threads - 1) / p.threads;
            if (p.cache_read >= 5) stage = 0;
            if (p.compute_at) stage = (bn * bk * es / 4 + p.threads - 1) / p.threads;
            if (p.compute_at == 3) {
                // only the helpers carry the patch, over 256 lanes
                int64_t rows = bm % op->OW == 0 ? bm / op->OW : (op->OW + bm - 2) / op->OW + 1;
                int64_t pr = (rows - 1) * d.stride + d.dilation * (d.dims[5] - 1) + 1, pw = (op->OW - 1) * d.stride + d.dilation * (d.dims[6] - 1) + 1;
                stage = std::max(stage, (pr * pw * d.dims[3] * es / 4 + 255) / 256);
            }
            if (p.compute_at == 2 && p.cache_read == 2) {
                // the next tile's patch waits in registers during the k loop
                int64_t rows = bm % op->OW == 0 ? bm / op->OW : (op->OW + bm - 2) / op->OW + 1;
                int64_t pr = (rows - 1) * d.stride + d.dilation * (d.dims[5] - 1) + 1, pw = (op->OW - 1) * d.stride + d.dilation * (d.dims[6] - 1) + 1;
                stage = std::max(stage, (pr * pw * d.dims[3] * es / 4 + p.threads - 1) / p.threads);
            }
            int64_t live = p.cache_read == 3 ? frag + 2 * stage : (p.cache_read >= 2 ? frag + stage : std::max(frag, stage));
            if (p.compute_at == 4) {
                // weight fragments of the wavefront's columns for every k step, A fragments of two steps
                int64_t fr = kp * es / 4 > 0 ? kp * es / 4 : 1;
                int64_t breg = (int64_t)p.tj[1] * p.tj[3] * ((int64_t)p.tk[0] * p.tk[1] * p.tk[2] * p.tk[3]) * fr; // every MFMA k step of the reduction
                int64_t areg = 2 * (int64_t)p.ti[1] * p.ti[3] * fr;
                int64_t pre = 0;
                if (p.cache_read == 2) {
                    int64_t rows = bm % op->OW == 0 ? bm / op->OW : (op->OW + bm - 2) / op->OW + 1;
                    int64_t pr = (rows - 1) * d.stride + d.dilation * (d.dims[5] - 1) + 1, pw = (op->OW - 1) * d.stride + d.dilation * (d.dims[6] - 1) + 1;
                    pre = (pr * pw * d.dims[3] * es / 4 + p.threads - 1) / p.threads;
                }
                int64_t have = 512 / ((p.waves + 3) / 4);
                if (breg + areg + pre + acc + 24 > have)
                    return reject("weights in registers: %" PRId64 " weight + %" PRId64 " operand + %" PRId64 " prefetch + %" PRId64
                                  " accumulator registers per lane exceed the %" PRId64 " a wavefront can have", breg, areg, pre, acc, have);
                frag = 0; // accounted for above
                stage = 0;
                live = 0;
            }
            if (p.cache_read == 4) {
                if (p.waves % 2) return reject("ping-pong wave groups need an even number of wavefronts, not %d", p.waves);
                if (p.tk[1] != 1 || p.tk[2] != 1) return reject("ping-pong wave groups need k1 = k2 = 1 (a tile's fragments are read in one phase)");
            }
            // a SIMD's 512 registers per lane are shared by the workgroup's wavefronts resident on it
            int64_t budget = 512 / ((p.waves + 3) / 4);
            // only the ping-pong schedule needs every fragment of a tile live at once; elsewhere the
            // compiler sequences the fragment reads, so the estimate is allowed to overshoot by half
            if (p.cache_read != 4) budget += budget / 2;
            if (live + acc > budget)
                return reject("%" PRId64 " fragment + %" PRId64 " staging + %" PRId64 " accumulator registers per lane exceed the %" PRId64
                              " a wavefront can have with %d wavefronts per workgroup", frag, stage, acc, budget, p.waves);
        } else if (p.cache_read) {
            int stages = p.cache_read;
            lds = (int64_t)stages * 4 * (bm * (bk + (p.lds_pad ? 4 : 0)) + bk * (bn + (p.lds_pad ? 4 : 0)));
            int64_t frag = ((int64_t)p.ti[1] * p.ti[3] + (int64_t)p.tj[1] * p.tj[3]) * p.tk[3];
            if (frag + acc > 448) return reject("%" PRId64 " operand + %" PRId64 " accumulator registers per lane exceed the register file", frag, acc);
        } else {
            if (p.lds_pad) return reject("storage_align without cache_read has nothing to pad");
            int64_t frag = ((int64_t)p.ti[1] * p.ti[3] + (int64_t)p.tj[1] * p.tj[3]) * p.tk[3];
            if (frag + acc > 448) return reject("%" PRId64 " operand + %" PRId64 " accumulator registers per lane exceed the register file", frag, acc);
        }
        if (lds > L.max_lds_bytes) return reject("LDS tile needs %" PRId64 " bytes, the limit is %d", lds, L.max_lds_bytes);
        p.lds_bytes = (int32_t)lds;
        // vectorize: alignment and divisibility of the global loads, per operand
        if (p.vec > 1) {
            int v = p.vec;
            if (v * es > 16) return reject("vector of %d x %d bytes is wider than a 16-byte load", v, es);
            if (is_conv2d(d.kind)) {
                if ((d.dims[3] / op->nb) % v) return reject("vector width %d does not divide Cin = %" PRId64 " (per group)", v, d.dims[3] / op->nb);
                if (bk % v) return reject("vector width %d does not divide the k tile %" PRId64, v, bk);
            } else {
                if (d.a_strides[2] != 1) return reject("vector loads of A need k contiguous");
                if (bk % v || d.a_strides[1] % v || (op->nb > 1 && d.a_strides[0] % v))
                    return reject("vector width %d breaks alignment of A (k tile %" PRId64 ", row stride %" PRId64 ")", v, bk, d.a_strides[1]);
            }
        }
        if (p.vec_b > 1) {
            int v = p.vec_b;
            if (v * es > 16) return reject("vector of %d x %d bytes is wider than a 16-byte load", v, es);
            if (is_conv2d(d.kind)) {
                if (op->N % v) return reject("vector width %d does not divide Cout = %" PRId64 " (per group)", v, op->N);
                if (bn % v) return reject("vector width %d does not divide the j tile %" PRId64, v, bn);
            } else if (d.b_strides[2] == 1) { // vector along j
                if (bn % v || d.b_strides[1] % v || (op->nb > 1 && d.b_strides[0] % v))
                    return reject("vector width %d breaks alignment of B (j tile %" PRId64 ", row stride %" PRId64 ")", v, bn, d.b_strides[1]);
            } else if (d.b_strides[1] == 1) { // vector along k
                if (bk % v || d.b_strides[2] % v || (op->nb > 1 && d.b_strides[0] % v))
                    return reject("vector width %d breaks alignment of B (k tile %" PRId64 ", column stride %" PRId64 ")", v, bk, d.b_strides[2]);
            } else {
                return reject("vector loads of B need j or k contiguous");
            }
        }
    } else if (space->family == MS_FAM_DWCONV) {
        if (!get_tile(space, trace, MS_SLOT_TILE_I, p.ti) || !get_tile(space, trace, MS_SLOT_TILE_J, p.tj) ||
            !get_tile(space, trace, MS_SLOT_TILE_C, p.tc))
            return fail(MS_ERR_BAD_ARG, "ms_trace_validate: the space lacks a tile slot");
        p.cache_read = (int32_t)cat_value(space, trace, MS_SLOT_CACHE_READ, 0);
        p.tile_unit[0] = p.tile_unit[1] = p.tile_unit[2] = 1;
        int64_t boh = (int64_t)p.ti[1] * p.ti[2] * p.ti[3], bow = (int64_t)p.tj[1] * p.tj[2] * p.tj[3],
                bc = (int64_t)p.tc[1] * p.tc[2] * p.tc[3];
        p.block_m = (int32_t)boh;
        p.block_n = (int32_t)bow;
        p.block_k = (int32_t)bc;
        int64_t threads = (int64_t)p.ti[2] * p.tj[2] * p.tc[2];
        if (threads > L.max_threads) return reject("%" PRId64 " threads per workgroup, the limit is %d", threads, L.max_threads);
        p.threads = (int32_t)threads;
        p.waves = (p.threads + L.wave_size - 1) / L.wave_size;
        // registers of one thread: the I3 x J3 output patch, its input patch and the taps, VC channels each
        int vc = p.tc[3] % 4 == 0 ? 4 : (p.tc[3] % 2 == 0 ? 2 : 1);
        int64_t patch_h = (int64_t)(p.ti[3] - 1) * d.stride + d.dims[4], patch_w = (int64_t)(p.tj[3] - 1) * d.stride + d.dims[5];
        int64_t acc = (int64_t)p.ti[3] * p.tj[3] * vc;
        int64_t regs = acc + (patch_h * patch_w + d.dims[4] * d.dims[5]) * vc;
        if (regs > L.max_acc_per_thread) return reject("%" PRId64 " registers for the output and input patch exceed the register budget %d", regs, L.max_acc_per_thread);
        p.acc_per_thread = (int32_t)acc;
        int64_t g = (int64_t)p.ti[0] * p.tj[0] * p.tc[0];
        if (g > 0x7fffffff / std::max<int64_t>(1, d.dims[0])) return reject("grid of %" PRId64 " workgroups overflows", g);
        p.grid[0] = (int32_t)g;
        p.grid[1] = 1;
        p.grid[2] = (int32_t)d.dims[0];
        p.vec = vc;
        if (p.cache_read) {
            int64_t ih = (boh - 1) * d.stride + d.dims[4], iw = (bow - 1) * d.stride + d.dims[5];
            int64_t lds = ih * iw * bc * 4;
            if (lds > L.max_lds_bytes) return reject("LDS halo tile needs %" PRId64 " bytes, the limit is %d", lds, L.max_lds_bytes);
            p.lds_bytes = (int32_t)lds;
        }
        p.tk[0] = 1;
        p.tk[1] = (int32_t)d.dims[4];
        p.tk[2] = (int32_t)d.dims[5];
        p.tk[3] = 1;
        p.unroll_k1 = p.unroll_k2 = p.unroll > 0 ? 0 : 1; // 0 = full unroll of the tap loops
    } else if (space->family == MS_FAM_REDUCE) {
        if (!get_tile(space, trace, MS_SLOT_TILE_I, p.ti) || !get_tile(space, trace, MS_SLOT_TILE_K, p.tk))
            return fail(MS_ERR_BAD_ARG, "ms_trace_validate: the space lacks a tile slot");
        p.cache_read = (int32_t)cat_value(space, trace, MS_SLOT_CACHE_READ, 0);
        if (d.kind == MS_OP_NORM) p.cache_read = 0; // a single pass anyway
        p.tile_unit[0] = p.tile_unit[1] = p.tile_unit[2] = 1;
        const int es = op->in_size;
        const int64_t k0 = p.tk[0], k1 = p.tk[1], k2 = p.tk[2], k3 = p.tk[3];
        if (k3 * es > 16 || (k3 & (k3 - 1))) return reject("vector of %" PRId64 " elements: a load moves 1, 2, 4, ... elements and at most 16 bytes", k3);
        if (op->out_size * k3 > 16) return reject("vector of %" PRId64 " output elements exceeds 16 bytes", k3);
        if (k2 > L.max_threads || (k2 & (k2 - 1))) return reject("%" PRId64 " lanes per row: the cross-thread reduction needs a power of two up to %d", k2, L.max_threads);
        if (d.kind == MS_OP_NORM && k2 < 64 && op->K > 4096)
            return reject("%" PRId64 " lanes would each sum %" PRId64 " squares in one fp32 chain; at least one wavefront per row", k2, op->K / k2);
        int64_t threads = (int64_t)p.ti[2] * k2;
        if (threads > L.max_threads) return reject("%" PRId64 " threads per workgroup, the limit is %d", threads, L.max_threads);
        if (threads % L.wave_size) return reject("%" PRId64 " threads per workgroup is not a whole number of wavefronts", threads);
        p.threads = (int32_t)threads;
        p.waves = p.threads / L.wave_size;
        if (k1 > 64) return reject("%" PRId64 " loads in flight per lane", k1);
        // values a lane holds at once: the rows of its group that are processed together, all of the lane's
        // share of them when the row stays in registers between the passes
        int64_t live = (int64_t)p.ti[3] * k1 * k3 * (p.cache_read ? k0 : 1);
        const int budget = std::min(L.max_acc_per_thread, 128); // the loaded vectors and the exponentials are live together
        if (live > budget) return reject("%" PRId64 " values per lane exceed the register budget %d", live, budget);
        if (p.cache_read && k0 * k1 > 64) return reject("%" PRId64 " loads per lane and row in a fully unrolled pass", k0 * k1);
        p.acc_per_thread = (int32_t)live;
        p.block_m = (int32_t)std::min<int64_t>((int64_t)p.ti[1] * p.ti[2] * p.ti[3], 0x7fffffff);
        p.block_n = 1;
        p.block_k = (int32_t)std::min<int64_t>(op->K, 0x7fffffff);
        p.vec = (int32_t)k3;
        p.grid[0] = p.ti[0];
        p.grid[1] = 1;
        p.grid[2] = 1;
        // partial results of the wavefronts of a group meet in LDS (maximum and sum use it in turn)
        p.lds_bytes = k2 > L.wave_size ? (int32_t)(p.waves * p.ti[3] * 4) : 0;
        p.unroll_k1 = (int32_t)k1;
        p.unroll_k2 = 1;
    } else {
        return fail(MS_ERR_BAD_ARG, "ms_trace_validate: unknown family %d", space->family);
    }
    if (!t_nests_only) resolve_body(op, &p);
    p.key = hash_params(op, &p);
    if (out) *out = p;
    return MS_OK;
}

// Estimate of a double-step launch in clocks: rounds of 256 persistent workgroups; a step is bound by the matrix cores, by its bytes
// from the L2 or by two barriers, and a tile starts and ends with nothing beside it.
static int64_t double_step_cost(const ms_op *op, const ms_variant_params *p, int64_t instances)
{
    const int64_t tiles = (int64_t)p->grid[0] * op->nb * instances, steps = op->K * op->in_size / 128, bm = p->block_m, bn = p->block_n;
    return (tiles + 255) / 256 * (2500 + steps * std::max<int64_t>({bm * bn / 24, (bm + bn) * 3, 600}) + bm * bn / 16);
}

bool ms::double_steps_few(const ms_op *op, const ms_variant_params *p, ms_variant_params *few)
{
    if (p->body != MS_BODY_DOUBLE_STEPS || op->M % 64 || op->N % 64 || g_limits.max_threads < 512 || g_limits.max_waves < 8) return false;
    *few = *p;
    set4(few->ti, op->M / 64, 1, 4, 1);
    set4(few->tj, op->N / 64, 1, 2, 2);
    few->block_m = few->block_n = 64;
    few->threads = 512;
    few->waves = 8;
    few->acc_per_thread = 8;
    if ((op->M / 64) * (op->N / 64) > 0x7fffffff / std::max<int64_t>(1, op->nb)) return false;
    few->grid[0] = few->ti[0] * few->tj[0];
    few->body_tile = double_steps(op, few);
    if (few->body_tile < 3) return false;
    few->lds_bytes = (int32_t)(few->body_tile * (int64_t)128 * 128 + double_step_staging(op, few));
    few->key = hash_params(op, few);
    return few->key != p->key && takes_few(op, p, few, 1);
}

bool ms::takes_few(const ms_op *op, const ms_variant_params *p, const ms_variant_params *few, int64_t instances)
{
    // not for what the estimate cannot tell.  768 x 576 x 2048 x 2 in bf16 (128 x 192 tiles on 24 compute units): 24.9 -> 12.8 us;
    // 576 x 1024 x 3264: 31.3 -> 18.4; 1024^3: 11.3 -> 8.5, x 2 stays at 11.3; 576 x 2048 x 1280, two rounds of 64 x 64, 15.4 and 16.6
    return double_step_cost(op, few, instances) * 10 < double_step_cost(op, p, instances) * 9;
}

bool ms::fill_kernel(const ms_op *op, const ms_variant_params *p, ms_variant_params *patch)
{
    if (p->family != MS_FAM_GEMM_MFMA) return false;
    if (op->d.kind == MS_OP_GEMM) {
        // not for what one instance does not take either; a split reduction is replaced too (128 x 1024 x 1024 in 8 parts, a second
        // kernel: 8.8 us and 3.3)
        const int tile = p->body == MS_BODY_NEST && op->M * op->N <= 1024 * 1024 ? few_rows(op) : 0;
        if (!tile) return false;
        const FewRows c = few_rows_tile(op, tile);
        *patch = *p;
        patch->body = MS_BODY_FEW_ROWS;
        patch->body_tile = tile;
        patch->block_m = c.mt * 16;
        patch->block_n = c.nc * 16;
        patch->block_k = c.waves * 32;
        patch->grid[0] = (int32_t)c.tiles;
        patch->grid[1] = patch->grid[2] = 1;
        patch->waves = c.waves;
        patch->threads = c.waves * 64;
        patch->acc_per_thread = c.mt * c.nc * 4;
        patch->lds_bytes = c.lds;
        patch->compute_at = patch->rfactor = patch->reorder = 0;
        patch->key = hash_params(op, patch);
        return true;
    }
    if (p->body == MS_BODY_IMAGE_ROWS) {
        const int tile = conv_planes(op);
        if (!tile) return false;
        const ConvPlanes c = conv_planes_tile(op, tile);
        *patch = *p;
        patch->body = MS_BODY_CONV_PLANES;
        patch->body_tile = tile;
        patch->body_tile_many = 0;
        patch->block_m = c.waves() * c.tm * 32;
        patch->grid[0] = (int32_t)c.tiles;
        patch->grid[1] = patch->grid[2] = 1;
        patch->waves = c.waves();
        patch->threads = c.waves() * 64;
        patch->acc_per_thread = c.tm * c.tn * 16;
        patch->lds_bytes = (int32_t)c.lds;
        patch->compute_at = 0;
        patch->reorder = 3;
        patch->key = hash_params(op, patch);
        return true;
    }
    const int tile = conv_patch(op);
    if (!tile) return false;
    const ConvPatch c = conv_patch_tile(op, tile);
    *patch = *p;
    patch->body = MS_BODY_CONV_PATCH;
    patch->body_tile = tile;
    patch->block_m = c.ws * c.wr * c.r * 16;
    patch->block_n = c.wj * c.tn * 16;
    patch->block_k = (int32_t)op->d.dims[5] * 32;
    patch->grid[0] = (int32_t)c.tiles;
    patch->grid[1] = patch->grid[2] = 1;
    patch->waves = c.waves + 1;
    patch->threads = patch->waves * 64;
    patch->acc_per_thread = c.r * c.tn * 4;
    patch->lds_bytes = (int32_t)c.lds;
    patch->compute_at = patch->rfactor = 0;
    patch->reorder = 3;
    patch->key = hash_params(op, patch);
    return true;
}

bool ms::takes_fill(const ms_op *op, const ms_variant_params *p, const ms_variant_params *patch, int64_t instances)
{
    if (patch->body == MS_BODY_FEW_ROWS) {
        // Up to 64 x 64 outputs per compute unit and four workgroups on each: there it is faster than the best of 60 to 120 sampled
        // nests (48 x 4096 x 2048: 7.0 us and 11.2; x 2: 10.5 and 12.2; 128 x 1024 x 1024: x 4 8.8 and 12.5; 128 x 8192 x 4096:
        // 23 and 33; 16 x 16384 x 4096: 23.1 and 23.5).  Beyond, nests fill the chip and load each operand fewer times (48 x 4096 x
        // 2048 x 8: 31 and 25; 16 x 1024 x 1024 x 64: 30 and 22; 128 x 16384 x 1024: 13.1 and 10.4).
        // Long reductions of few tiles that the trace splits over workgroups keep its nest, second kernel included: tiles leave half of the chip
        // idle (16 x 3072 x 4096: 11.3 us and 9.2; 32 x 1280 x 4096: 9.9 and 8.1; 32 x 2048 x 4096: 9.3 and 8.7).  Up to 64 tiles the
        // weights are read from the caches (32 x 1024 x 4096: 5.2 and 9.2; 16 x 2048 x 4096: 9.7 and 9.9), shorter reductions and more rows
        // lose by the partial sums (16 x 4096 x 3072: 8.5 and 8.8; 32 x 2048 x 3072: 7.2 and 7.6; 48 x 1344 x 4096: 8.2 and 8.9).
        const int64_t tiles = patch->grid[0] * instances;
        if (p->rfactor >= 4 && tiles > 64 && tiles <= 128 && op->K >= 2560 + 48 * op->M) return false;
        return tiles <= 1024 && op->M * op->N * instances <= 1024 * 1024;
    }
    if (patch->body == MS_BODY_CONV_PLANES) {
        // Launches whose rounds leave more than a quarter of the chip idle spread better in the smaller tiles of image rows (3 x 16 x
        // 64 x 64 -> 64, 7 x 7 x 7, x 4: 11.5 us and 18.7); two rounds of tiles of 3 x 2 intrinsics whose second one is less than two
        // thirds full do so too (128 x 128 x 3 -> 64, 7 x 7, batch 75, 825 of 1024: 12.2 and 13.7; 192 x 192 x 3 -> 64, 7 x 7, batch 36, 864:
        // 14.8 and 14.1; 4 x 2, 192 x 192 x 3 -> 64, 7 x 7, batch 47, 846: 20.4 and 18.2).  A single round hides no loads under small tiles
        // (64 x 64 x 4 -> 64, 7 x 7, batch 114: 7.4 and 8.1) or large ones of few steps (192 x 192 x 4 -> 64, 3 x 3, batch 27: 9.3 and 10.1).
        const ConvPlanes c = conv_planes_tile(op, patch->body_tile);
        const int64_t tiles = (int64_t)patch->grid[0] * instances, slots = 256 * c.per_cu(), busy = (tiles + slots - 1) / slots * slots;
        if (c.tn == 1) return tiles * 100 >= busy * 75;
        if (tiles <= slots && (c.tm < 3 || (c.tm == 4 && op->kd == 1 && c.steps < 4))) return false;
        return tiles * 100 >= busy * (c.tm <= 3 && busy == 2 * slots ? 83 : 75);
    }
    // its wavefronts count steps in 32 bits
    const int64_t tiles = (int64_t)patch->grid[0] * instances;
    if (tiles * op->K > 0x7fffffffll * 256 || (instances > 1 && !(patch->body_tile & CONV_PATCH_MANY))) return false;
    // The tiles of a batch that would run on gathers are as large as these and lose to them at any size (28 x 28 x 128 -> 128,
    // batch 4: 10.3 us and 9.2, batch 64: 21.4 and 17.3).  Elsewhere the last round must not leave too much of the chip idle: 35 % of
    // the rounds' workgroups have to be there where single images would run on gathers (28 x 28 x 128 -> 128 x 32, 64 tiles: 22 and
    // 26; x 128: 69 and 27), 60 % for nests of small tiles (16 x 16 x 64 -> 64, batch 330: 23.3 and 14.7; 40 x 40 x 96 -> 32 x 80: 33
    // and 17), 80 % for those whose weights and patches stay in LDS too (56 x 56 x 64 -> 64, four tiles: x 1 7.8 and 15.5, x 32 15.7 and
    // 17.7, x 64 22.7 and 20.0, x 80 27.1 and 29.4, x 200 57.6 and 59.4).
    const int64_t slots = 256 * fill_per_cu(op, patch), busy = (tiles + slots - 1) / slots * slots;
    const bool gathers = p->body == MS_BODY_CONV_STEPS, single = op->d.dims[0] == 1;
    return (gathers && !single) || tiles * 100 >= busy * (gathers ? 35 : p->compute_at >= 2 && single ? 80 : 60);
}

int ms::fill_per_cu(const ms_op *op, const ms_variant_params *p)
{
    return p->body == MS_BODY_CONV_PLANES ? conv_planes_tile(op, p->body_tile).per_cu() : conv_patch_tile(op, p->body_tile).per_cu;
}

int32_t ms::validate_as_nest(const ms_op *op, const ms_space *space, const ms_trace *trace, ms_variant_params *out)
{
    t_nests_only = true;
    const int32_t rc = ms_trace_validate(op, space, trace, out);
    t_nests_only = false;
    return rc;
}

namespace ms {

static std::string def(const char *name, int64_t v)
{
    char buf[96];
    snprintf(buf, sizeof buf, "-D%s=%" PRId64, name, v);
    return buf;
}

static int dt_code(int32_t dt) { return dt; }

// the -D options of the loop nest that the factors spell out
static void push_schedule(std::vector<std::string> &D, const ms_variant_params *p)
{
    const char *tn[4] = {"I", "J", "C", "K"};
    const int32_t *tl[4] = {p->ti, p->tj, p->tc, p->tk};
    for (int l = 0; l < 4; ++l)
        for (int f = 0; f < 4; ++f) {
            char nm[8];
            snprintf(nm, sizeof nm, "%s%d", tn[l], f);
            D.push_back(def(nm, tl[l][f] ? tl[l][f] : 1));
        }
    D.push_back(def("NTHREADS", p->threads));
    D.push_back(def("CACHE_READ", p->cache_read));
    D.push_back(def("VEC", p->vec));
    D.push_back(def("VEC_B", p->vec_b > 0 ? p->vec_b : 1));
    D.push_back(def("CACHE_WRITE", p->cache_write));
    D.push_back(def("UNROLL_K1", p->unroll_k1));
    D.push_back(def("UNROLL_K2", p->unroll_k2));
    D.push_back(def("LDS_PAD", p->lds_pad));
    D.push_back(def("REORDER", p->reorder));
    D.push_back(def("COMPUTE_AT", p->compute_at));
    D.push_back(def("HELPER_WAVES", p->compute_at == 3 ? 4 : 0));
    D.push_back(def("RFACTOR", p->rfactor > 1 ? p->rfactor : 1));
}

int32_t make_kernel_spec(const ms_op *op, const ms_variant_params *p, KernelSpec *out)
{
    const ms_op_desc &d = op->d;
    KernelSpec k;
    k.entry = "ms_kernel";
    k.block[0] = (unsigned)p->threads;
    k.block[1] = k.block[2] = 1;
    k.grid[0] = (unsigned)p->grid[0];
    k.grid[1] = (unsigned)p->grid[1];
    k.grid[2] = (unsigned)p->grid[2];
    k.lds_dynamic = 0;
    k.many_grid = 0;
    auto &D = k.defines;
    D.push_back(def("IN_DT", dt_code(d.in_dtype)));
    D.push_back(def("OUT_DT", dt_code(d.out_dtype)));
    const bool conv_patch = p->body == MS_BODY_CONV_PATCH, conv_steps = p->body == MS_BODY_CONV_STEPS;
    if (follows_decisions(p) || conv_steps) push_schedule(D, p);
    if (p->family == MS_FAM_GEMM_ALU || p->family == MS_FAM_GEMM_MFMA) {
        D.push_back(def("DIM_B", op->nb));
        D.push_back(def("DIM_M", op->M));
        D.push_back(def("DIM_N", op->N));
        D.push_back(def("DIM_K", conv_steps ? op->K / conv_steps_tile(op, p->block_m, p->block_n).phases : op->K));
        bool conv = is_conv2d(d.kind) && !conv_steps && !conv_patch;
        D.push_back(def("IS_CONV", conv ? 1 : 0));
        if (conv) {
            D.push_back(def("CV_N", d.dims[0]));
            D.push_back(def("CV_H", d.dims[1]));
            D.push_back(def("CV_W", d.dims[2]));
            D.push_back(def("CV_CIN", d.dims[3] / op->nb)); // channels a group reduces over
            D.push_back(def("CV_XC", d.dims[3]));           // channels per pixel of X
            D.push_back(def("CV_COUT", d.dims[4]));
            D.push_back(def("LDC", d.dims[4]));             // output channels per pixel of Y = bias values per instance
            D.push_back(def("C_BATCH", op->N));             // a group's outputs start op->N channels after the previous group's
            D.push_back(def("CV_KH", d.dims[5]));
            D.push_back(def("CV_KW", d.dims[6]));
            D.push_back(def("CV_OH", op->OH));
            D.push_back(def("CV_OW", op->OW));
            D.push_back(def("CV_STRIDE", d.stride));
            D.push_back(def("CV_PAD", d.pad));
            D.push_back(def("CV_PAD_H", op->pad_h));
            D.push_back(def("CV_D", op->depth));
            D.push_back(def("CV_KD", op->kd));
            D.push_back(def("CV_OD", op->OD));
            D.push_back(def("CV_DIL", d.dilation));
            D.push_back(def("CV_TRANSPOSED", d.kind == MS_OP_CONV2D_TRANSPOSED_NHWC ? 1 : 0));
            if (follows_decisions(p)) {
                if (d.kind == MS_OP_CONV2D_TRANSPOSED_NHWC) D.push_back(def("CV_PHASES", p->body == MS_BODY_PHASES ? 1 : 0));
                D.push_back(def("CV_TAPROWS", p->tap_rows));
                D.push_back(def("CV_KR", (d.dims[6] * d.dims[3] + p->tile_unit[2] - 1) / p->tile_unit[2] * p->tile_unit[2]));
            }
            D.push_back(def("HAS_BIAS", d.has_bias ? 1 : 0));
            D.push_back(def("RELU", d.relu ? 1 : 0));
            // implicit GEMM view: A rows are output pixels, B = W as [K][N]
            D.push_back(def("SA_B", d.dims[3] / op->nb)); // channel offset of a group
            D.push_back(def("SA_I", 0));
            D.push_back(def("SA_K", 1));
            D.push_back(def("SB_B", op->N));              // column offset of a group in W [K][Cout]
            D.push_back(def("SB_K", d.dims[4]));
            D.push_back(def("SB_J", 1));
            D.push_back(def("A_INST", d.dims[0] * op->depth * d.dims[1] * d.dims[2] * d.dims[3]));
            D.push_back(def("B_INST", op->K * op->N * op->nb));
        } else if (conv_steps || conv_patch) {
            const bool transposed = d.kind == MS_OP_CONV2D_TRANSPOSED_NHWC;
            const int64_t S = transposed ? d.stride : 1;
            if (conv_steps) {
                D.push_back(def("CONV_STEPS", 1));
                D.push_back(def("PP_STAGES", conv_steps_tile(op, p->block_m, p->block_n).stages));
            }
            D.push_back(def("HAS_BIAS", d.has_bias ? 1 : 0));
            D.push_back(def("RELU", d.relu ? 1 : 0));
            D.push_back(def("CS_TR", transposed ? 1 : 0));
            D.push_back(def("CS_N", d.dims[0]));
            D.push_back(def("CS_H", d.dims[1]));
            D.push_back(def("CS_W", d.dims[2]));
            D.push_back(def("CS_C", d.dims[3]));
            D.push_back(def("CS_KW", d.dims[6]));
            D.push_back(def("CS_TH", d.dims[5] / S));
            D.push_back(def("CS_TW", d.dims[6] / S));
            D.push_back(def("CS_S", d.stride));
            D.push_back(def("CS_DIL", std::max(1, (int)d.dilation)));
            D.push_back(def("CS_PAD_H", op->pad_h));
            D.push_back(def("CS_PAD_W", d.pad));
            D.push_back(def("CS_PN", S));
            D.push_back(def("CS_PH_H", op->OH / S));
            D.push_back(def("CS_PH_W", op->OW / S));
            D.push_back(def("SA_B", 0));
            D.push_back(def("SA_I", 0));
            D.push_back(def("SA_K", 1));
            D.push_back(def("SB_B", 0));
            D.push_back(def("SB_K", op->N));
            D.push_back(def("SB_J", 1));
            D.push_back(def("A_INST", d.dims[0] * d.dims[1] * d.dims[2] * d.dims[3]));
            D.push_back(def("B_INST", op->K * op->N));
        } else {
            D.push_back(def("HAS_BIAS", 0));
            D.push_back(def("RELU", 0));
            D.push_back(def("SA_B", d.a_strides[0]));
            D.push_back(def("SA_I", d.a_strides[1]));
            D.push_back(def("SA_K", d.a_strides[2]));
            D.push_back(def("SB_B", d.b_strides[0]));
            D.push_back(def("SB_K", d.b_strides[1]));
            D.push_back(def("SB_J", d.b_strides[2]));
            int64_t ab, bb;
            ms_op_tensor_bytes(op, 0, &ab);
            ms_op_tensor_bytes(op, 1, &bb);
            D.push_back(def("A_INST", ab / op->in_size));
            D.push_back(def("B_INST", bb / op->in_size));
        }
        if (p->body == MS_BODY_FEW_ROWS) {
            const FewRows c = few_rows_tile(op, p->body_tile);
            k.template_name = "gemm_rows.hip";
            D.push_back(def("FR_MT", c.mt));
            D.push_back(def("FR_NC", c.nc));
            D.push_back(def("FR_WAVES", c.waves));
            D.push_back(def("FR_DEPTH", c.depth));
            D.push_back(def("FR_LDS", c.lds));
        } else if (conv_patch) {
            const ConvPatch c = conv_patch_tile(op, p->body_tile);
            k.template_name = "conv_patch.hip";
            D.push_back(def("CP_CW", c.cw));
            D.push_back(def("CP_R", c.r));
            D.push_back(def("CP_TN", c.tn));
            D.push_back(def("CP_WR", c.wr));
            D.push_back(def("CP_WJ", c.wj));
            D.push_back(def("CP_WHOLE", c.whole));
            D.push_back(def("CP_THREADS", (c.waves + 1) * 64));
            D.push_back(def("CP_PER_CU", c.per_cu));
            D.push_back(def("CP_LDS", c.lds));
        } else if (p->body == MS_BODY_CONV_PLANES) {
            const ConvPlanes c = conv_planes_tile(op, p->body_tile);
            k.template_name = "conv_planes.hip";
            D.push_back(def("CR_TM", c.tm));
            D.push_back(def("CR_TN", c.tn));
            D.push_back(def("CR_WAVES", c.waves()));
            D.push_back(def("CR_LDS", c.lds));
        } else if (p->body == MS_BODY_IMAGE_ROWS) {
            const ConvRows cr = conv_rows_tiles(op, p->body_tile);
            k.template_name = "conv_rows.hip";
            D.push_back(def("CR_TM", cr.tm));
            D.push_back(def("CR_TN", cr.tn));
            D.push_back(def("CR_SPAN", cr.tpr ? 1 : 0));
            D.push_back(def("CR_WAVES", p->waves));
            if (p->body_tile_many) {
                const ConvRows many = conv_rows_tiles(op, p->body_tile_many);
                D.push_back(def("CR_MANY_TM", many.tm));
                D.push_back(def("CR_MANY_SPAN", many.tpr ? 1 : 0));
                k.many_grid = (unsigned)many.groups;
            }
        } else if (p->family == MS_FAM_GEMM_MFMA) {
            k.template_name = "gemm_mfma.hip";
            D.push_back(def("MI_M", p->tile_unit[0]));
            D.push_back(def("MI_N", p->tile_unit[1]));
            D.push_back(def("MI_K", p->tile_unit[2]));
            if (p->body == MS_BODY_DOUBLE_STEPS) D.push_back(def("PP_STAGES", p->body_tile));
        } else {
            k.template_name = "gemm_alu.hip";
        }
    } else if (p->family == MS_FAM_REDUCE) {
        k.template_name = "reduce.hip";
        D.push_back(def("RD_OP", d.kind == MS_OP_NORM ? 1 : 0));
        D.push_back(def("RD_ROWS", op->M));
        D.push_back(def("RD_LEN", op->K));
        if (p->body == MS_BODY_ROW_VECTORS) {
            D.push_back(def("ROW_VEC", p->body_tile));
            D.push_back(def("ROW_LANES", p->tk[2]));
            D.push_back(def("ROW_WAVES", p->waves));
        }
    } else {
        k.template_name = "dwconv.hip";
        D.push_back(def("CV_N", d.dims[0]));
        D.push_back(def("CV_H", d.dims[1]));
        D.push_back(def("CV_W", d.dims[2]));
        D.push_back(def("CV_C", d.dims[3]));
        D.push_back(def("CV_KH", d.dims[4]));
        D.push_back(def("CV_KW", d.dims[5]));
        D.push_back(def("CV_OH", op->OH));
        D.push_back(def("CV_OW", op->OW));
        D.push_back(def("CV_STRIDE", d.stride));
        D.push_back(def("CV_PAD", d.pad));
        if (p->body == MS_BODY_STRIPS) {
            D.push_back(def("STRIP", p->body_tile));
            D.push_back(def("STRIP_THREADS", p->threads));
        }
    }
    *out = k;
    return MS_OK;
}

} // namespace ms

bool ms::image_rows_many(const ms_op *op, const ms_variant_params *p, int64_t instances, int64_t *lds)
{
    if (p->body != MS_BODY_IMAGE_ROWS || !p->body_tile_many || instances < 2) return false;
    const ConvRows few = conv_rows_tiles(op, p->body_tile), many = conv_rows_tiles(op, p->body_tile_many);
    if (lds) *lds = many.lds;
    // short reductions (filters below 7 x 7 x 3) are bound by the launch's first loads and last stores: four full rounds, or the
    // larger tile gains nothing (112 x 112 x 3 -> 64, 3 x 3, stride 2 x 64: 8.3 us with tm = 1, 9.9 with 4; 224 x 224 x 4 -> 64,
    // 3 x 3 x 64: 118 and 96)
    if (many.steps * op->kd < 11 && many.groups * instances < 4 * many.slots()) return false;
    return many.cost(instances) < few.cost(instances);
}

extern "C" int32_t ms_variant_kernel_text(const ms_op *op, const ms_variant_params *p, char *buf, size_t cap, size_t *needed)
{
    if (!op || !p) return fail(MS_ERR_BAD_ARG, "ms_variant_kernel_text: NULL argument");
    KernelSpec k;
    int32_t rc = make_kernel_spec(op, p, &k);
    if (rc != MS_OK) return rc;
    std::string s = k.template_name + "\n";
    for (auto &d : k.defines) s += d + "\n";
    if (needed) *needed = s.size() + 1;
    if (buf && cap) {
        size_t n = std::min(cap - 1, s.size());
        memcpy(buf, s.data(), n);
        buf[n] = 0;
    }
    return MS_OK;
}

// Phase form of the transposed convolution: output row of tile i0's row lr, filter taps that meet a phase.
static int64_t phase_out_row(const ms_op *op, const ms_variant_params *p, int64_t i0, int64_t lr)
{
    const int64_t S = op->d.stride, ph_h = op->OH / S, ph_w = op->OW / S, cls = i0 % (S * S), u = i0 / (S * S) * p->block_m + lr;
    return (u / (ph_h * ph_w) * op->OH + u / ph_w % ph_h * S + cls / S) * op->OW + u % ph_w * S + cls % S;
}
static int64_t phase_tap(int64_t ph, int64_t pad, int64_t S, int64_t t) { return (ph + pad) % S + S * t; }

// Index of the four-level split: ((x0*f1 + x1)*f2 + x2)*f3 + x3.
static inline int64_t split_index(const int32_t *f, int64_t x0, int64_t x1, int64_t x2, int64_t x3)
{
    return ((x0 * f[1] + x1) * f[2] + x2) * f[3] + x3;
}

extern "C" int32_t ms_variant_coverage(const ms_op *op, const ms_variant_params *p, int32_t *counts, int64_t out_elems)
{
    if (!op || !p || !counts) return fail(MS_ERR_BAD_ARG, "ms_variant_coverage: NULL argument");
    int64_t ob;
    ms_op_tensor_bytes(op, -1, &ob);
    if (out_elems != ob / op->out_size) return fail(MS_ERR_BAD_ARG, "ms_variant_coverage: out_elems %" PRId64 " != %" PRId64, out_elems, ob / op->out_size);
    memset(counts, 0, sizeof(int32_t) * (size_t)out_elems);
    const ms_op_desc &d = op->d;
    if (p->body == MS_BODY_IMAGE_ROWS) {
        const ConvRows c = conv_rows_tiles(op, p->body_tile);
        const int64_t bn = c.tn * 32, jbs = op->N / bn, ohw = op->OH * op->OW;
        for (int64_t wg = 0; wg < c.groups; ++wg) {
            const int64_t jb = wg % jbs, od = wg / jbs % op->OD, tile = wg / (jbs * op->OD) % c.tiles, n = wg / (jbs * op->OD * c.tiles);
            const int64_t oh = c.tpr ? tile / c.tpr : 0, first = c.tpr ? oh * op->OW + tile % c.tpr * c.px : tile * c.px;
            const int64_t end = c.tpr ? (oh + 1) * op->OW : ohw;
            for (int64_t px = first; px < first + c.px; ++px)
                for (int64_t j = 0; j < bn; ++j) {
                    if (px >= end) continue; // pixels behind the plane, or the row, are not stored
                    const int64_t at = ((n * op->OD + od) * ohw + px) * op->N + jb * bn + j;
                    if (at >= out_elems) return fail(MS_ERR_INVALID_TRACE, "coverage: index out of range");
                    ++counts[at];
                }
        }
    } else if (p->body == MS_BODY_CONV_STEPS) {
        const ConvSteps c = conv_steps_tile(op, p->block_m, p->block_n);
        const int64_t S = d.kind == MS_OP_CONV2D_TRANSPOSED_NHWC ? d.stride : 1, rows = op->M / c.phases;
        for (int64_t wg = 0; wg < p->grid[0]; ++wg) {
            const int64_t i0 = wg / p->tj[0], j0 = wg % p->tj[0];
            for (int64_t lr = 0; lr < c.bm; ++lr) {
                if (i0 / c.phases * c.bm + lr >= rows) continue; // pixels behind the last one are not stored
                const int64_t i = S == 1 ? i0 * c.bm + lr : phase_out_row(op, p, i0, lr);
                for (int64_t j = 0; j < c.bn; ++j) {
                    const int64_t at = i * op->N + j0 * c.bn + j;
                    if (at >= out_elems) return fail(MS_ERR_INVALID_TRACE, "coverage: index out of range");
                    ++counts[at];
                }
            }
        }
    } else if (p->body == MS_BODY_STRIPS) {
        const int64_t C = d.dims[3], strip = p->body_tile, sw = p->tj[0];
        for (int64_t n = 0; n < d.dims[0]; ++n)
            for (int64_t item = 0; item < (int64_t)p->grid[0] * p->threads; ++item) {
                if (item >= (int64_t)p->ti[0] * sw * C) continue;
                const int64_t ch = item % C, ow = item / C % sw * strip, oh = item / (C * sw) * strip;
                for (int64_t a = 0; a < strip; ++a)
                    for (int64_t b = 0; b < strip; ++b)
                        if (oh + a < op->OH && ow + b < op->OW) ++counts[((n * op->OH + oh + a) * op->OW + ow + b) * C + ch];
            }
    } else if (p->family == MS_FAM_GEMM_ALU || p->family == MS_FAM_GEMM_MFMA) {
        int um = p->tile_unit[0], un = p->tile_unit[1];
        for (int64_t b = 0; b < op->nb; ++b)
            for (int64_t wg = 0; wg < p->grid[0] / std::max(1, p->rfactor); ++wg) { // output tiles (rfactor workgroups share one)
                int64_t i0, j0;
                if (p->reorder == 1) {
                    j0 = wg / p->ti[0];
                    i0 = wg % p->ti[0];
                } else {
                    i0 = wg / p->tj[0];
                    j0 = wg % p->tj[0];
                }
                for (int64_t t = 0; t < (int64_t)p->ti[2] * p->tj[2]; ++t) { // thread or wavefront
                    int64_t ti = t / p->tj[2], tj = t % p->tj[2];
                    for (int64_t r1 = 0; r1 < p->ti[1]; ++r1)
                        for (int64_t r3 = 0; r3 < p->ti[3]; ++r3)
                            for (int64_t c1 = 0; c1 < p->tj[1]; ++c1)
                                for (int64_t c3 = 0; c3 < p->tj[3]; ++c3) {
                                    int64_t iu = split_index(p->ti, i0, r1, ti, r3);
                                    int64_t ju = split_index(p->tj, j0, c1, tj, c3);
                                    for (int a = 0; a < um; ++a)
                                        for (int c = 0; c < un; ++c) {
                                            int64_t i = iu * um + a, j = ju * un + c;
                                            if (p->body == MS_BODY_PHASES) i = phase_out_row(op, p, i0, i - i0 * p->block_m);
                                            if (i >= op->M || j >= op->N) return fail(MS_ERR_INVALID_TRACE, "coverage: index out of range");
                                            if (is_conv2d(op->d.kind)) ++counts[i * (op->N * op->nb) + b * op->N + j]; // groups interleave per pixel
                                            else ++counts[(b * op->M + i) * op->N + j];
                                        }
                                }
                }
            }
    } else if (p->family == MS_FAM_REDUCE) {
        const bool per_element = op->d.kind == MS_OP_SOFTMAX, masked = p->body == MS_BODY_ROW_VECTORS;
        for (int64_t wg = 0; wg < p->grid[0]; ++wg)
            for (int64_t r1 = 0; r1 < p->ti[1]; ++r1)
                for (int64_t g = 0; g < p->ti[2]; ++g)
                    for (int64_t r3 = 0; r3 < p->ti[3]; ++r3) {
                        int64_t row = split_index(p->ti, wg, r1, g, r3);
                        if (masked && row >= op->M) continue;
                        if (row >= op->M) return fail(MS_ERR_INVALID_TRACE, "coverage: index out of range");
                        if (!per_element) {
                            ++counts[row];
                            continue;
                        }
                        for (int64_t q0 = 0; q0 < p->tk[0]; ++q0)
                            for (int64_t q1 = 0; q1 < p->tk[1]; ++q1)
                                for (int64_t t = 0; t < p->tk[2]; ++t)
                                    for (int64_t q3 = 0; q3 < p->tk[3]; ++q3) {
                                        int64_t k = split_index(p->tk, q0, q1, t, q3);
                                        if (masked && k >= op->K) continue;
                                        if (k >= op->K) return fail(MS_ERR_INVALID_TRACE, "coverage: index out of range");
                                        ++counts[row * op->K + k];
                                    }
                    }
    } else {
        int64_t C = d.dims[3];
        for (int64_t n = 0; n < d.dims[0]; ++n)
            for (int64_t wg = 0; wg < p->grid[0]; ++wg) {
                int64_t c0 = wg % p->tc[0], j0 = wg / p->tc[0] % p->tj[0], i0 = wg / ((int64_t)p->tc[0] * p->tj[0]);
                for (int64_t t = 0; t < p->threads; ++t) {
                    int64_t tc = t % p->tc[2], tj = t / p->tc[2] % p->tj[2], ti = t / ((int64_t)p->tc[2] * p->tj[2]);
                    for (int64_t r1 = 0; r1 < p->ti[1]; ++r1)
                        for (int64_t r3 = 0; r3 < p->ti[3]; ++r3)
                            for (int64_t q1 = 0; q1 < p->tj[1]; ++q1)
                                for (int64_t q3 = 0; q3 < p->tj[3]; ++q3)
                                    for (int64_t s1 = 0; s1 < p->tc[1]; ++s1)
                                        for (int64_t s3 = 0; s3 < p->tc[3]; ++s3) {
                                            int64_t oh = split_index(p->ti, i0, r1, ti, r3);
                                            int64_t ow = split_index(p->tj, j0, q1, tj, q3);
                                            int64_t c = split_index(p->tc, c0, s1, tc, s3);
                                            if (oh >= op->OH || ow >= op->OW || c >= C) return fail(MS_ERR_INVALID_TRACE, "coverage: index out of range");
                                            ++counts[((n * op->OH + oh) * op->OW + ow) * C + c];
                                        }
                }
            }
    }
    return MS_OK;
}

extern "C" int32_t ms_variant_reduction_coverage(const ms_op *op, const ms_variant_params *p, int32_t *counts, int64_t k_elems, int64_t *needed)
{
    if (!op || !p) return fail(MS_ERR_BAD_ARG, "ms_variant_reduction_coverage: NULL argument");
    const bool dw = p->family == MS_FAM_DWCONV;
    const int unit = dw ? 1 : std::max(1, p->tile_unit[2]);
    const bool masked = p->body == MS_BODY_ROW_VECTORS || p->body == MS_BODY_IMAGE_ROWS || p->body == MS_BODY_CONV_STEPS; // positions beyond K are left out
    const int64_t len = dw ? (int64_t)op->d.dims[4] * op->d.dims[5] : masked ? op->K : (int64_t)p->tk[0] * p->tk[1] * p->tk[2] * p->tk[3] * unit;
    if (needed) *needed = len;
    if (!counts) return needed ? MS_OK : fail(MS_ERR_BAD_ARG, "ms_variant_reduction_coverage: NULL argument");
    if (k_elems != len) return fail(MS_ERR_BAD_ARG, "ms_variant_reduction_coverage: k_elems %" PRId64 " != %" PRId64, k_elems, len);
    // the interpreted reduction covers the operator's K, padded by less than one intrinsic where a convolution rounds it up
    if (!dw && !masked && !p->tap_rows && (len < op->K || len - op->K >= unit))
        return fail(MS_ERR_INVALID_TRACE, "reduction coverage: the split covers %" PRId64 " positions, the operator reduces over %" PRId64, len, op->K);
    memset(counts, 0, sizeof(int32_t) * (size_t)len);
    if (dw) {
        for (int64_t kh = 0; kh < p->tk[1]; ++kh)
            for (int64_t kw = 0; kw < p->tk[2]; ++kw) {
                int64_t k = kh * op->d.dims[5] + kw;
                if (k >= len) return fail(MS_ERR_INVALID_TRACE, "reduction coverage: index out of range");
                ++counts[k];
            }
        return MS_OK;
    }
    if (p->body == MS_BODY_IMAGE_ROWS) {
        // per filter plane the chunks of its runs; elements before and behind a run are masked
        const ConvRows c = conv_rows_tiles(op, p->body_tile);
        const int64_t KH = op->d.dims[5], run = op->d.dims[6] * op->d.dims[3];
        for (int64_t kd = 0; kd < op->kd; ++kd)
            for (int64_t ch = 0; ch < c.steps * 2; ++ch)
                for (int64_t e = 0; e < 8; ++e) {
                    const int64_t q = ch % c.cpr * 8 + e - c.lead;
                    if (ch < KH * c.cpr && q >= 0 && q < run) ++counts[(kd * KH + ch / c.cpr) * run + q];
                }
        return MS_OK;
    }
    if (p->body == MS_BODY_CONV_STEPS) {
        // every output phase walks its own taps; together they are the filter
        const ms_op_desc &d = op->d;
        const ConvSteps c = conv_steps_tile(op, p->block_m, p->block_n);
        const int64_t S = d.kind == MS_OP_CONV2D_TRANSPOSED_NHWC ? d.stride : 1, cin = d.dims[3];
        for (int64_t cls = 0; cls < c.phases; ++cls)
            for (int64_t k = 0; k < c.steps * 64; ++k) {
                if (k >= c.th * c.tw * cin) continue;
                const int64_t t = k / cin, kh = S == 1 ? t / c.tw : phase_tap(cls / S, op->pad_h, S, t / c.tw), kw = S == 1 ? t % c.tw : phase_tap(cls % S, d.pad, S, t % c.tw);
                const int64_t at = (kh * d.dims[6] + kw) * cin + k % cin;
                if (at < 0 || at >= len) return fail(MS_ERR_INVALID_TRACE, "reduction coverage: index out of range");
                ++counts[at];
            }
        return MS_OK;
    }
    const int rf = std::max(1, p->rfactor);
    if (p->tk[0] % rf) return fail(MS_ERR_INVALID_TRACE, "reduction coverage: rfactor does not divide k0");
    if (p->body == MS_BODY_PHASES) {
        // every output phase walks its own taps; together they are the filter
        const ms_op_desc &d = op->d;
        const int64_t S = d.stride, cin = d.dims[3], tw = d.dims[6] / S, steps = p->tk[0] / (S * S), bk = p->block_k;
        for (int64_t cls = 0; cls < S * S; ++cls)
            for (int64_t k = 0; k < steps * bk; ++k) {
                const int64_t t = k / cin, kh = phase_tap(cls / S, op->pad_h, S, t / tw), kw = phase_tap(cls % S, d.pad, S, t % tw);
                const int64_t at = (kh * d.dims[6] + kw) * cin + k % cin;
                if (at < 0 || at >= len) return fail(MS_ERR_INVALID_TRACE, "reduction coverage: index out of range");
                ++counts[at];
            }
        return MS_OK;
    }
    const int64_t run = p->tk[0] / rf; // k0 steps of one workgroup
    for (int64_t s = 0; s < rf; ++s)
        for (int64_t q0 = s * run; q0 < (s + 1) * run; ++q0)
            for (int64_t q1 = 0; q1 < p->tk[1]; ++q1)
                for (int64_t q2 = 0; q2 < p->tk[2]; ++q2)
                    for (int64_t q3 = 0; q3 < p->tk[3]; ++q3)
                        for (int u = 0; u < unit; ++u) {
                            int64_t k = split_index(p->tk, q0, q1, q2, q3) * unit + u;
                            if (masked && k >= len) continue;
                            if (k < 0 || k >= len) return fail(MS_ERR_INVALID_TRACE, "reduction coverage: index out of range");
                            ++counts[k];
                        }
    return MS_OK;
}
