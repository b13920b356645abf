// Host-side logic: argument validation, launch plan, buffer sizes, status strings.
#include <initializer_list>

#include "cg_common.h"

namespace cg {

static int validate_desc(const codegemm_desc* d)
{
    if (!d) return CODEGEMM_INVALID_ARG;
    if (d->batch < 1 || d->in_features < 1 || d->out_features < 1) return CODEGEMM_INVALID_ARG;
    if (d->vec_len != 4 && d->vec_len != 8 && d->vec_len != 16) return CODEGEMM_UNSUPPORTED;
    if (d->num_codebooks < 1 || d->num_codebooks > 4) return CODEGEMM_UNSUPPORTED;
    if (d->code_bits != 8) return CODEGEMM_UNSUPPORTED;
    // Every byte offset the kernels form (a workgroup's code range, a row of x) stays below 2^31.
    if (d->batch > kMaxBatch || d->in_features > kMaxInFeatures || d->out_features > kMaxOutFeatures)
        return CODEGEMM_UNSUPPORTED;
    if (d->in_features % d->vec_len) return CODEGEMM_INVALID_ARG;
    if (d->group_size != -1) {
        // one scale per g = v * 2^i weights, groups tiling K exactly
        const int g = d->group_size;
        if (g < d->vec_len || g % d->vec_len) return CODEGEMM_UNSUPPORTED;
        const int ratio = g / d->vec_len;
        if (ratio & (ratio - 1)) return CODEGEMM_UNSUPPORTED;
        if (d->in_features % g) return CODEGEMM_INVALID_ARG;
    }
    if (d->flags & ~CODEGEMM_FLAG_Y_FP32) return CODEGEMM_INVALID_ARG;
    return CODEGEMM_OK;
}

// Formats the centroid kernel takes: a group of scales covers at least what one MFMA contracts over (4 chunks: 4
// sub-vectors, 8 for v = 4), and the codes of a step fit in registers.
static bool centroid_format(const codegemm_desc* d)
{
    if (d->vec_len == 4 && d->num_codebooks > 2) return false;
    return d->group_size == -1 || d->group_size >= (d->vec_len == 4 ? 8 : 4) * d->vec_len;
}

// Batch rows of a workgroup of the centroid kernel whose blocks have `rows` rows.  A wavefront owns 32, 64 or 128
// rows and takes 4, 8 or 16 batch rows per MFMA; blocks lower than the batch would have take several MFMAs per lookup.
static int centroid_batch(const codegemm_desc* d, int rows)
{
    const int b = d->batch;
    if (b <= 8) return b == 1 ? 1 : b <= 4 ? 4 : 8;
    // two tiles of 16 only where their accumulators leave registers for the codes
    const bool two = d->group_size == -1 && !(d->flags & CODEGEMM_FLAG_Y_FP32) && ((d->vec_len == 8 && d->num_codebooks <= 2) || (d->vec_len == 4 && d->num_codebooks == 1));
    return b > 16 && rows == 128 && two ? 32 : 16;
}
// Groups shorter than a step of the kernels (16 chunks) flush their sums inside it, with more registers.
static bool short_groups(const codegemm_desc* d)
{
    return d->group_size > 0 && (d->group_size < (d->vec_len == 4 ? 32 : 16) * d->vec_len || (d->flags & CODEGEMM_FLAG_Y_FP32));
}
// Formats that the kernel with staged operands has (gemm_staged_impl.h).
static bool staged_format(const codegemm_desc* d)
{
    return !(d->flags & CODEGEMM_FLAG_Y_FP32) && ((d->vec_len == 8 && d->num_codebooks <= 2) || (d->vec_len == 4 && d->num_codebooks == 1));
}
static int centroid_min_rows(const codegemm_desc* d)
{
    if (staged_format(d)) return 32;
    if (d->vec_len < 16) {
        if (d->batch <= 8 || d->num_codebooks == 1) return 32;
        if (d->group_size < 0) return d->flags & CODEGEMM_FLAG_Y_FP32 ? 64 : 32;
        return short_groups(d) ? 128 : 64;                                                     // registers
    }
    return d->batch <= 4 ? 32 : d->batch <= 8 ? 64 : 128;      // v = 16: one MFMA per lookup (registers)
}

// Batch rows of a workgroup of the kernel that stages codes and x in LDS, or 0: the centroid kernel.  `range` is the K of a workgroup.  Measured on 59 000 random sizes under every block height
// and 1 to 8 K ranges, time of the centroid kernel / time here, by range, up to 256 workgroups (above: the centroid kernel has two workgroups on
// a compute unit, the rings leave room for one):
//  * 2 to 4 rows: 128-row blocks with group scales, where the centroid kernel picks one result element of four and scales it: v8 m1 1.10 at 2048,
//    1.21 at 5000, 1.38 at 12000 (above 256 workgroups 0.81 at 1500, 0.91, 1.03, 1.17); v8 m2 1.03, 1.12, 1.20 (0.77, 0.86, 0.92, 1.01); v4 m1 1.02, 1.07,
//    1.14 (0.78, 0.89, 0.95, 1.01).  The lines are 3072, 4096 and 7168.  Without group scales 0.9 to 1.07 (v8 m1 1.2 from 8192 on), and lower blocks
//    lose at any K but the longest (64 rows 0.83 to 1.02, v8 m1 with group scales 1.16; 32 rows 0.8 to 0.97): there the centroid kernel's 16
//    columns are all at work, and its rings hold a whole short slice.
//  * 5 to 8 rows: 32-row blocks v8 m2 1.06 to 1.31, others 1.0 to 1.18; 64-row blocks 1.01 to 1.28; 128-row blocks v8 m2 1.10 to 1.19, v8 m1 with
//    group scales 1.12 to 1.40, without 1.05, 1.00, 1.06, 1.13, 1.29 (0.86 and 0.93 at 1500 and 3000, 1.00 at 6000, 1.19): from 8192 on; v4 m1 1.03, 1.08,
//    1.13, 1.22, 1.36 (0.88, 0.90, 0.97, 1.07): from 2048 on, and so with group scales.
//  * 9 to 32 rows: 32-row blocks 1.2 to 2.0, 64-row blocks 1.14 to 1.8, 128-row blocks 1.1 to 1.4: a lookup there pays one MFMA for 16 rows at any
//    height, where the centroid kernel's columns are octets x sub-vectors and take two or four.  17 to 32 rows are two tiles of 16 in one
//    workgroup but for v8 m1, and 128-row blocks with group scales (registers): one tile per workgroup; v8 m1 has no such 128-row kernel.
//  * Groups of 4 and 8 chunks, which take a scaled sum per round either way (12 000 other sizes): 32-row blocks 1.1 to 1.25 at 5 to 8 rows and 1.3 to 1.7
//    beyond, 64-row blocks 1.2 to 1.4 and 1.7 to 2.9 (the centroid kernel spills there), 128-row blocks 1.05 to 1.3 and 1.25 to 1.4; v8 m1 has no 128-row
//    kernel (47 registers of spills).
// It does not depend on the number of workgroups: a layer alone has others than in a group.
static int staged_batch(const codegemm_desc* d, int rows, int range)
{
    const int v = d->vec_len, m = d->num_codebooks, b = d->batch;
    const bool grouped = d->group_size > 0, wide = v == 8 && m == 1;
    if (!staged_format(d)) return 0;
    if (b <= 4) return rows == 128 && b > 1 && !short_groups(d) && grouped && range >= (v == 4 ? 7168 : wide ? 3072 : 4096) ? 4 : 0;
    if (rows < 128) return b <= 8 ? 8 : b <= 16 || wide ? 16 : 32;
    if (b <= 8 && range < (v == 4 ? 2048 : grouped ? 0 : wide ? 8192 : 1024)) return 0;
    if (wide && grouped) return b <= 8 && !short_groups(d) ? 8 : 0;
    if (wide && b <= 16 && range < 2048) return 0;
    if (b <= 16 || grouped) return 16;
    return wide ? 0 : 32;
}

// Batch rows of a workgroup of whichever of the two runs.  Above kBatchPerLaunch rows, where a layer has no group to agree with, two tiles of 16
// become workgroups of their own while these are one round: half of the work each in place of an idle half of the chip (6232->2777 v4 m1, 73
// rows, 64-row blocks: 132 workgroups 16.4 us, 220 13.0).
static int batch_rows(const codegemm_desc* d, int rows, int splits, bool* is_staged = nullptr)
{
    const int nkt = ceil_div(d->in_features / d->vec_len, kSlots), units = ceil_div(nkt, splits < nkt ? splits : nkt);
    int staged = staged_batch(d, rows, units * kSlots * d->vec_len);
    if (staged == 32 && d->batch > kBatchPerLaunch && (long long)ceil_div(d->out_features, rows) * ceil_div(d->batch, 16) * ceil_div(nkt, units) <= 256) staged = 16;
    if (is_staged) *is_staged = staged != 0;
    return staged ? staged : centroid_batch(d, rows);
}

// 2 to 4 rows with group scales: blocks of 128 rows in two or four K ranges on the staged kernel instead of lower ones on the
// centroid kernel, where these fill the chip and leave every workgroup a long K (3200 random sizes, 160 to 256 workgroups, time
// here / of the lower blocks at 4096, 6144, 8192, 10240 and 12288 elements per workgroup: v8 m1 0.99, 0.92, 0.88, 0.85, 0.83; v8 m2 1.03, 0.98,
// 0.94, 0.93, 0.91; v4 m1 1.08 to 1.0: left out).  It belongs to the choice of the default plan: a group's members and their
// layers alone then follow the same fields, and a plan that asks for lower blocks gets them.
static void raise_to_staged(const codegemm_desc* d, codegemm_plan* p)
{
    if (p->centroid_rows == 128 || d->batch < 2 || d->vec_len != 8 || d->group_size < 0) return;
    const long long blocks = ceil_div(d->out_features, kGranuleRows);
    const int splits = 4 * blocks <= 256 ? 4 : 2, nkt = ceil_div(d->in_features / d->vec_len, kSlots);
    if (d->batch > 4 || splits * blocks < 160 || splits * blocks > 256 || splits > p->k_splits || splits > nkt) return;
    const int range = ceil_div(nkt, splits) * kSlots * d->vec_len;
    if (range < (d->num_codebooks == 1 ? 6144 : 7168) || !staged_batch(d, kGranuleRows, range)) return;
    p->centroid_rows = kGranuleRows;
    p->centroid_splits = splits;
}

// A plan made for one batch, output type or format of a layer serves the others too, as its Psumbook fields do: blocks
// become as high as this problem's registers and grid ask for, and where the centroid kernel does not take the format
// the Psumbook fields hold, and so they do for an fp16 Psumbook.  There are no more K ranges than k_splits, and than the
// ticket counters and, above kBatchPerLaunch rows, the partial sums of a launch of that many rows have room for.
void resolve_centroid(const codegemm_desc* d, long long n, codegemm_plan* p)
{
    if (p->centroid_rows == 0) return;
    int rows = p->centroid_rows > centroid_min_rows(d) ? p->centroid_rows : centroid_min_rows(d);
    auto blocks = [&]() { return (n + rows - 1) / rows; };
    while (rows < 128 && blocks() > kMaxRowBlocks) rows *= 2;
    if (!centroid_format(d) || p->psum_dtype == CODEGEMM_PSUM_FP16 || blocks() > kMaxRowBlocks) {
        p->centroid_rows = p->centroid_splits = 0;
        return;
    }
    p->centroid_rows = rows;
    if (p->centroid_splits > p->k_splits) p->centroid_splits = p->k_splits;
    const long long groups = ceil_div(d->batch, centroid_batch(d, rows));
    if ((blocks() + kMaxGroup - 1) * groups > kCounterAreaWords) p->centroid_splits = 1;
}

static int validate_plan(const codegemm_desc* d, const codegemm_plan* p)
{
    if (p->waves != 8 && p->waves != 14 && p->waves != 16) return CODEGEMM_UNSUPPORTED;
    if (p->waves == 14) {
        // 448-row blocks: gather kernel for one or two batch rows only, fp32 Psumbook, registers as for 16 wavefronts
        if (p->row_words != 2 || p->batch_group > 2 || p->psum_dtype != CODEGEMM_PSUM_FP32) return CODEGEMM_UNSUPPORTED;
    }
    if (p->row_words != 1 && p->row_words != 2 && p->row_words != 4) return CODEGEMM_UNSUPPORTED;
    if (p->row_words == 4 && p->waves != 16 && p->batch_group != 4) return CODEGEMM_UNSUPPORTED;
    if (p->k_splits < 1) return CODEGEMM_UNSUPPORTED;
    if (p->batch_group != 1 && p->batch_group != 2 && p->batch_group != 4) return CODEGEMM_UNSUPPORTED;
    if (p->centroid_rows == 0) {
        if (p->centroid_splits != 0) return CODEGEMM_INVALID_ARG;
    } else {
        if (p->centroid_rows != 32 && p->centroid_rows != 64 && p->centroid_rows != 128) return CODEGEMM_INVALID_ARG;
        if (p->centroid_splits < 1) return CODEGEMM_INVALID_ARG;
    }
    if (p->build_waves != 0 && p->build_waves != 2) return CODEGEMM_UNSUPPORTED;
    if (p->build_waves == 2) {
        // 14 gathering + 2 building wavefronts: a double-buffered fp32 Psumbook (one or two codebooks); one batch
        // row per pass with two row words, or the batched kernel with one or two
        if (p->waves != 16 || p->psum_dtype != CODEGEMM_PSUM_FP32 || d->num_codebooks > 2) return CODEGEMM_UNSUPPORTED;
        if (p->batch_group == 1 ? p->row_words != 2 : (p->batch_group != 4 || p->row_words > 2)) return CODEGEMM_UNSUPPORTED;
    }
    if (p->psum_dtype != CODEGEMM_PSUM_FP32 && p->psum_dtype != CODEGEMM_PSUM_FP16) return CODEGEMM_UNSUPPORTED;
    if (p->psum_dtype == CODEGEMM_PSUM_FP16) {
        if (p->batch_group != 1 || p->row_words > 2) return CODEGEMM_UNSUPPORTED;
        if (d->group_size > 0 && p->waves == 16 && p->row_words == 2) return CODEGEMM_UNSUPPORTED;   // registers
        return CODEGEMM_OK;
    }
    const int m = d->num_codebooks;
    if (p->batch_group == 4) {
        // the batched kernel: 32 accumulators per row word
        if (p->row_words == 4 && p->waves != 8) return CODEGEMM_UNSUPPORTED;
        return CODEGEMM_OK;
    }
    if (p->row_words >= 2 && p->batch_group * m > (p->waves == 8 ? 8 : 4)) return CODEGEMM_UNSUPPORTED;   // accumulators + code ring must fit in registers
    if (p->row_words == 4 && (p->batch_group != 1 || m > 2 || d->group_size > 0)) return CODEGEMM_UNSUPPORTED;
    return CODEGEMM_OK;
}

// Library's own choice.  One workgroup per compute unit is resident (its Psumbook
// buffers take 128 KB of LDS).  A workgroup must stream about 32 KB of codes per K tile
// to keep up with its share of HBM, so blocks are 512 rows tall when the batch and the
// number of codebooks leave registers for it; the K ranges are then cut to give close
// to, but not more than, 256 workgroups.
static void choose_psumbook_plan(const codegemm_desc* d, codegemm_plan* p)
{
    *p = codegemm_plan{};
    const int m = d->num_codebooks;
    const int J = d->in_features / d->vec_len;
    const int ngr = ceil_div(d->out_features, kGranuleRows);
    const int nkt = ceil_div(J, kSlots);
    const double code_positions = (double)d->out_features * J;
    // Two batch rows: the batch-1 kernel with the code words reused for a second Psumbook, except on
    // large matrices, where the batched kernel wins even with two of its four batch lanes idle
    // (8192->28672: 32.7 -> 25.6 us; 8192^2: 11.4 against 12.0)
    const int batch = d->batch < kBatchPerLaunch ? d->batch : kBatchPerLaunch;
    p->batch_group = batch == 1 ? 1 : ((batch == 2 && code_positions < 16e6) ? 2 : 4);
    if (p->batch_group == 4) {
        // LDS- and ALU-bound.  Every workgroup rebuilds the Psumbook of its tiles, and LDS
        // writes are slow, so blocks are 1024 rows tall when there are at least two batch
        // groups to fill the chip with, 512 otherwise; K ranges are cut so that all batch
        // groups together give close to, but not more than, 256 workgroups.
        const int groups = ceil_div(batch, 4);
        auto fill = [&](int waves, int row_words, int* k_splits) {      // workgroups of a block shape
            const int nblk = ceil_div(ngr * kGranuleRows, waves * row_words * 32) * groups;
            int nks = 256 / nblk;
            if (nks > nkt) nks = nkt;
            if (nks < 1) nks = 1;
            *k_splits = ceil_div(nkt, ceil_div(nkt, nks));
            return nblk * *k_splits;
        };
        p->waves = 16;
        p->row_words = groups >= 2 ? 2 : 1;
        if (groups == 1) {
            // one batch group: 1024-row blocks only if every workgroup still gets 4 units of K
            // from at most 16 K ranges
            // (8192->28672 at batch 4: 32.4 -> 27.5 us; with 1 unit each they lose: 13.0 -> 16.6)
            const int nblk2 = ceil_div(ngr, 8);
            int nks2 = 256 / nblk2;
            if (nks2 > nkt) nks2 = nkt;
            if (nks2 < 1) nks2 = 1;
            if (ceil_div(nkt, nks2) >= 4 && nks2 <= 16) p->row_words = 2;   // (28 ranges: 30.1 -> 32.7 us)
        }
        // The 1024-row shape with 16 wavefronts has 128 registers per lane: with group scales, or
        // three and more codebooks, its 64 accumulators and the scale ring no longer fit and it
        // spills (8192->28672, m2v8g128, batch 8: 93 us against 56 us with 512-row blocks).
        if (p->row_words == 2 && (d->group_size > 0 || m >= 3)) p->row_words = 1;
        // Small matrices: a shorter block when the taller one leaves most of the chip idle
        // (2048^2 at batch 8: 32 workgroups of 1024 rows 19.5 us, 128 of 256 rows 7.8 us).
        int ks = 1;
        int wgs = fill(p->waves, p->row_words, &ks);
        if (wgs < 192 && p->row_words == 2) {
            int ks1 = 1;
            const int w1 = fill(16, 1, &ks1);
            if (w1 > wgs) { p->row_words = 1; wgs = w1; ks = ks1; }
        }
        if (wgs < 192 || ks > 32) {
            // also when the chip is only filled by cutting K into more than 32 ranges: the last
            // workgroup of a row block then adds that many partial sums per output
            // (8192->2048, v4 m1, batch 4: 64 ranges 13.2 us)
            int ks8 = 1;
            const int w8 = fill(8, 1, &ks8);
            if (w8 > wgs || (w8 >= 192 && ks8 < ks)) { p->waves = 8; p->row_words = 1; wgs = w8; ks = ks8; }
        }
        p->k_splits = ks;
        // Heights that 448 (896) rows divide, one or two codebooks: 14 of the 16 wavefronts own the rows
        // and 2 build every tile's Psumbook one tile ahead; the blocks then also fill 256 compute units
        // where 512 (1024) rows give 224 (4096->14336 v8 m2, batch 4 / 8 / 16 / 32: -5 / -9 / -12 / -11 %;
        // 8192->28672 m2v8g128 batch 4 / 8: -9 / -10 %).  With a ragged last block it loses (8192 rows: +10 %).
        if (p->waves == 16 && m <= 2) {
            const int rows = 14 * p->row_words * 32;
            const int nblk14 = ceil_div(d->out_features, rows);
            if ((long long)nblk14 * rows * 50 <= (long long)ngr * kGranuleRows * 51) {        // at most 2 % of padding
                int ks14 = 1;
                const int wgs14 = fill(14, p->row_words, &ks14);
                if (wgs14 >= wgs && wgs14 >= 192) {
                    p->k_splits = ks14;
                    p->build_waves = 2;
                }
            }
        }
        return;
    }
    // 512-row blocks for large matrices with up to three codebooks, 256-row blocks (more, shorter
    // K ranges; twice the registers per lane) otherwise -- from plan sweeps on the Llama-3 shapes
    p->waves = (code_positions >= 16e6 && p->batch_group * m <= 4) ? 16 : 8;
    p->row_words = (p->batch_group * m <= (p->waves == 8 ? 8 : 4)) ? 2 : 1;
    // K ranges: as many as give close to, but not more than, 256 workgroups (one per compute
    // unit).  When K is too short for that with 2 row words, blocks of half the height double
    // the workgroups (plan sweeps: 1024-output shapes -0.3 us).
    auto ranges = [&](int row_words, int* workgroups) {
        const int nblk = ceil_div(ngr * kGranuleRows, row_words * p->waves * 16);
        int nks = 256 / nblk;
        if (nks > nkt) nks = nkt;
        if (nks < 1) nks = 1;
        nks = ceil_div(nkt, ceil_div(nkt, nks));          // no empty K range
        *workgroups = nblk * nks;
        return nks;
    };
    int wgs = 0;
    p->k_splits = ranges(p->row_words, &wgs);
    // 448-row blocks (14 wavefronts) when they fill more of the 256 compute units: heights of
    // 7 * 2^k rows (the Llama up/gate projections) divide into 224 workgroups of 512 rows but
    // into 256 of 448.  Measured at 8192->28672: -2 % to -5 % for one and three codebooks and with
    // group scales; with two or four codebooks and one scale per row a tie or a loss (+0.1 us),
    // because the 8m MFMA blocks of a Psumbook then divide evenly over 16 wavefronts and not over 14.
    // With one or two codebooks the 448 rows go to 14 of 16 wavefronts and the other two build
    // every Psumbook, one unit ahead (build_waves = 2), when a workgroup has at least four units
    // to stream: 8192->28672 v8 m1 10.0 -> 9.8 us, v4 m1 15.3 -> 14.0, v4 m1 g128 19.3 -> 17.0,
    // m2v8g128 15.6 -> 15.2 against the 14-wavefront shape (two codebooks, one scale per row: 14.5 both).
    if (p->waves == 16 && p->row_words == 2 && ((m & 1) || d->group_size > 0)) {
        p->waves = 14;
        int wgs14 = 0;
        const int nks14 = ranges(2, &wgs14);
        if (wgs14 > wgs && wgs >= 192) {
            p->k_splits = nks14;
            if (m <= 2 && ceil_div(nkt, nks14) >= 4) {
                p->waves = 16;
                p->build_waves = 2;
            }
            return;
        }
        p->waves = 16;
    }
    if (p->row_words == 2 && wgs <= 128) {
        int wgs1 = 0;
        const int nks1 = ranges(1, &wgs1);
        if (wgs1 > wgs) {
            p->row_words = 1;
            p->k_splits = nks1;
        }
    }
}

// Rows of a block of the centroid kernel for up to 4 batch rows: as low as one round of 256 workgroups allows.  A second
// round that few blocks are left for costs as much as a full one: 257 to 320 blocks of 32 rows take 1.09 to 1.42 times as
// long as half as many of 64 rows, 257 to 448 of 64 rows 1.04 to 1.35 times as long as of 128 (random sizes, all formats).
static int low_rows(int n) { return ceil_div(n, 32) <= 256 ? 32 : ceil_div(n, 64) <= 256 ? 64 : 128; }

// Whether the centroid kernel is the faster one, from 61 000 random sizes at up to 4 batch rows, 43 000 at 5 to 32 and
// 17 000 above (times: Psumbook kernels / centroid kernel).  Its cost is the lookups of one workgroup, rows times K of a
// block, four times the LDS bytes of the Psumbook's; the Psumbook kernels cut K finer and fill the chip at any height.
//  * One row: where that work is small.  Ratio at 32-row blocks on more than half of the chip (64 rows: at half the K,
//    128 at a quarter): v8 m2 1.2 at K = 2000, 1.1 at 4000, 1.1 at 7000, 1.0 at 16000; v8 m1 1.2, 1.2, 1.15, 1.05; v4 m1
//    (the shortest centroids) 1.3, 1.3, 1.25, 1.2, below 1 from 128-row blocks with K = 8000 on unless a step lies in
//    one group.  8192^2 v8 m2 ties and is left out.  fp32 output of v8 m2 group scales: half of the work; with one scale
//    per row it gains nothing.  v8 group scales tie below K = 1024; three codebooks and v = 16 lose.
//  * Two to four rows: everywhere (v8 m2, 2 / 4 rows: 1.4 / 1.7; v4 m1 1.5 / 1.8), but for v8 with group scales or fp32
//    output on blocks of 64 and 128 rows that fill less than three quarters of the chip, from a work of 128 x 8192 on
//    (two rows, v8 m1 g128: 0.75 to 0.97 at K = 8300 to 28000 and 16400 to 18000 rows), and v16 with three or four codebooks, whose lookups read 32
//    bytes (two rows, v16 m4: 1.2 below K = 4000, 0.95 to 1.05 at 8000, 0.8 to 0.9 from 16000 on).
//  * Groups shorter than a step cost a flush inside it.  With several codebooks the register-loading kernel has only 128-row
//    blocks for them from nine rows on, too few of them on small matrices (v8 m3 and fp32 output below 4 million codes), and v = 16 loses at two
//    rows.  v8 m2 with fp16 output has staged blocks of 32 rows at any size (2400 random sizes of 30 000 to 1.1 million codes, g 32 and 64, 9 to 32
//    rows, Psumbook / staged kernel: 1.31 to 2.61, 1.74 in the mean; 2048^2 g32, 9, 16 and 32 rows: 7.5/4.6, 7.8/4.7 and 10.5/5.9 us).
//  * fp32 output pays for its short chains of sums: v = 16 loses on small matrices, at two rows (m2 8192^2 8.4/9.4) and
//    with three and four codebooks, and above 8 rows its 16 products per sum leave it less exact than the Psumbook
//    kernels (1.04 to 1.08 of their error below K = 8192).
//  * 5 to 32 rows: v16 on small matrices (0.76 to 0.97; m4 at batch 16: 4096^2 14.8/16.0, 8192^2 31.7/20.6), blocks of v8
//    that are too few when they have to be 128 rows (group scales: up to 1100 rows; fp32 output: 1500), and short K with
//    fp32 output above 16 rows.  The staged kernel's blocks of 32 rows are enough of them at any height (v8 m2 g128, batch 16,
//    Psumbook / staged: 1024 rows of K = 8192 13.0/5.7 us, 1100 of 4096 10.6/5.3).
//  * More: everywhere (33 to 64 rows 2.4, to 128 3.2, to 512 4.4, to 2048 6 and more; no size of 17 000 lost 1 %).
static bool prefer_centroid(const codegemm_desc* d)
{
    if (!centroid_format(d) || d->out_features > kMaxRowBlocks * 128) return false;
    const int v = d->vec_len, m = d->num_codebooks, batch = d->batch, K = d->in_features, N = d->out_features;
    const bool fp32 = d->flags & CODEGEMM_FLAG_Y_FP32, grouped = d->group_size > 0;
    const long long codes = (long long)m * N * (K / v);
    if (short_groups(d)) {
        if (batch > 8 && batch <= kBatchPerLaunch && m > 1 && !staged_format(d) && codes < 4000000) return false;
        if (v == 16 && batch == 2 && m > 2) return false;
    }
    if (fp32 && v == 16 && (batch > 8 || codes < 6000000 || batch == 2 || m > 2)) return false;
    if (batch > kBatchPerLaunch) return true;
    if (batch <= 4) {
        const int rows = low_rows(N), nb = ceil_div(N, rows);
        const long long work = (long long)rows * K;
        if (batch == 1) {
            if (m > 2 || v == 16 || (fp32 && !grouped && m > 1)) return false;
            if (v == 4 && m == 1) return (N >= 4096 || K >= 8192) && ((grouped && !short_groups(d)) || work < 32 * 24576);
            if (N < 4096 || (grouped && v == 8 && K < 1024)) return false;
            if (m == 1) return work <= 32 * 12288;
            return K < 8192 && work <= 32 * (fp32 ? 4096 : 8192);
        }
        if (v == 16) return m < 3 || work <= (nb >= 192 ? 128 * 8192 : batch == 2 ? 64 * 4096 : 64 * 8192);
        if (v == 8 && nb < 192 && (grouped || fp32)) return work <= 128 * (batch > 2 ? 14336 : fp32 || m == 1 ? 8192 : 16384);
        return true;
    }
    const int n64 = ceil_div(N, 64);
    if (v == 16) {
        if (m >= 3 && (batch <= 8 ? n64 <= 64 : batch < 24 && codes < 10000000)) return false;
        return batch <= 8 || codes >= (batch <= 16 ? 6000000 : 4000000);
    }
    if (batch > 8 && v == 8 && m >= 2 && !staged_format(d) && (grouped ? n64 <= 18 : fp32 && n64 < 24)) return false;
    return !(batch > 16 && fp32 && K < 1024);
}

// Microseconds of a call of 5 rows and more in blocks of `rows` rows and `splits` K ranges, for the formats of the staged kernel: a fixed part
// per call and round of 256 workgroups, a workgroup's K at a rate per format, batch and height, and the exchange between the ranges (two and
// four pairwise where their words fit, else by the ticket).  A round that is not full streams faster (what bounds it is the chip's power): a
// quarter of the stream's time follows the workgroups and not the rounds.  Fitted to 17 000 random sizes of 5 to 700 rows that are no prompts, under
// every height and 1, 2, 3, 4, 6 and 8 ranges; the spread about it is 9 %.  On 9000 other sizes the plans that it leads to take 1.006 (5 to 8 rows), 1.005
// (9 to 16), 1.011 (17 to 32) and 1.007 (more) of the time of the best of these plans, the rules of choose_plan alone 1.010, 1.027, 1.066 and 1.054.
// Short groups: rates of 11 000 sizes of their own, the other numbers the same; 1.003, 1.004 and 1.011 (17 and more), the rules 1.032, 1.094 and 1.071.
static float batch_cost(const codegemm_desc* d, int rows, int splits)
{
    // us per 1024 elements of K: [v4 m1, v8 m1, v8 m2][one scale per row, groups that hold a step, short groups][up to 8, 16, more rows][blocks of
    // 32, 64, 128 rows]
    static const float rates[3][3][3][3] = {
        {{{0.57f, 0.99f, 1.46f}, {0.76f, 1.18f, 1.64f}, {1.60f, 1.95f, 2.81f}},
         {{0.62f, 1.08f, 1.70f}, {0.76f, 1.13f, 1.69f}, {1.34f, 1.66f, 1.50f}},
         {{0.67f, 1.15f, 1.90f}, {0.85f, 1.28f, 1.85f}, {1.47f, 1.92f, 1.69f}}},
        {{{0.49f, 0.66f, 1.14f}, {0.64f, 0.83f, 1.23f}, {0.64f, 0.76f, 3.31f}},
         {{0.56f, 0.76f, 1.18f}, {0.68f, 0.87f, 1.92f}, {0.66f, 0.78f, 1.64f}},
         {{0.61f, 0.93f, 2.56f}, {0.72f, 1.03f, 2.62f}, {0.73f, 0.92f, 2.21f}}},
        {{{0.69f, 1.17f, 1.78f}, {0.81f, 1.27f, 1.84f}, {1.59f, 2.12f, 3.64f}},
         {{0.77f, 1.36f, 2.32f}, {1.29f, 1.41f, 2.36f}, {1.83f, 2.15f, 2.05f}},
         {{0.81f, 1.35f, 2.45f}, {0.93f, 1.44f, 2.50f}, {1.60f, 2.39f, 2.28f}}}};
    // us: a call, a round, the exchange of two and of four ranges pairwise, and of any number by the ticket
    static const float call[3] = {1.24f, 1.28f, 1.56f};
    static const float round[3][3] = {{2.53f, 2.49f, 3.21f}, {2.47f, 2.65f, 3.45f}, {2.33f, 2.87f, 3.97f}};
    static const float two[3][3] = {{0.61f, 0.65f, 0.91f}, {0.71f, 0.79f, 1.06f}, {0.85f, 0.90f, 1.33f}};
    static const float four[3][3] = {{1.08f, 1.14f, 1.59f}, {1.20f, 1.42f, 1.77f}, {1.37f, 1.55f, 2.07f}};
    static const float ticket[3][3] = {{1.97f, 1.99f, 3.08f}, {2.10f, 2.94f, 4.30f}, {2.97f, 3.81f, 5.85f}};
    const bool wide = d->vec_len == 8 && d->num_codebooks == 1;
    const int b = d->batch, tile = batch_rows(d, rows, splits), h = rows == 32 ? 0 : rows == 64 ? 1 : 2;
    // (v8 m1, and 128-row blocks with group scales, have the rates of two tiles of 16 rows in the last column)
    const int c = b <= 8 ? 0 : b <= 16 || (b > kBatchPerLaunch && tile == 16 && !wide && (rows < 128 || d->group_size < 0)) ? 1 : 2;
    const int nkt = ceil_div(d->in_features / d->vec_len, kSlots);
    const int units = ceil_div(nkt, splits < nkt ? splits : nkt), range = units * kSlots * d->vec_len;
    splits = ceil_div(nkt, units);
    const long long workgroups = (long long)ceil_div(d->out_features, rows) * ceil_div(b, tile) * splits;
    const float rounds = (float)((workgroups + 255) / 256), full = (float)workgroups * (1.0f / 256);
    const bool pairs = (splits == 2 || splits == 4) &&
                       (long long)b * (splits - 1) * ceil_div(d->out_features, kGranuleRows) * kGranuleRows * 8 <= (long long)kPairAreaBytes;
    // (more than 8 ranges were not timed: 0.1 us each, as the batched kernel's ticket takes)
    const float exchange = splits == 1 ? 0.0f : pairs ? (splits == 2 ? two : four)[c][h] : ticket[c][h] + 0.1f * (float)(splits > 8 ? splits - 8 : 0);
    const float stream = rates[d->vec_len == 4 ? 0 : d->num_codebooks][short_groups(d) ? 2 : d->group_size > 0][c][h] * (float)range * (1.0f / 1024);
    return call[c] + rounds * round[c][h] + (0.73f * rounds + 0.27f * full) * stream + exchange;
}

static void choose_plan(const codegemm_desc* d, codegemm_plan* p)
{
    choose_psumbook_plan(d, p);
    if (!prefer_centroid(d)) return;
    const int nkt = ceil_div(d->in_features / d->vec_len, kSlots);
    const long long codes = (long long)d->num_codebooks * d->out_features * (d->in_features / d->vec_len);
    const int least = centroid_min_rows(d);
    auto blocks = [&](int r) { return (long long)ceil_div(d->out_features, r) * ceil_div(d->batch, centroid_batch(d, r)); };
    // Block height.  Low blocks need fewer K ranges, and with them the exchange through memory; from 5 batch rows on
    // they cost the register-loading kernel more MFMAs per lookup (32 rows: one per 4 batch rows, 64: one per 8).  So: as low as fills the chip, and
    // only for matrices whose lookups are few beside a call's fixed part.  (The staged formats, whose low blocks pay one MFMA at any height, only start
    // from this choice: the costs below have the last word.  Times of the register-loading kernel, v8 m2, us: batch 8, 2048^2 32 rows 5.6, 64 rows
    // 6.6; 4096^2 6.5 / 7.8; 8192^2 13.6 / 11.1; batch 16, 4096^2 32 rows 9.0, 64 rows 9.5, 128 rows 11.3; 4096->14336
    // 64 rows 12.5, 128 rows 14.0; 14336->4096 17.0 / 14.0; batch 32, 4096^2 64 rows 10.5, 128 rows 15.8).
    int rows = 128;
    if (d->batch <= 4) {
        rows = low_rows(d->out_features);
        // 513 to 768 blocks of 64 rows, two or three on a compute unit, where those of 128 rows are staged, one on a unit, and take a second round
        // (700 random sizes, 2 to 4 rows, time of 64 rows / of 128 staged / of 128 on the centroid kernel, in parts of the second: v8 m1 0.87 / 1 / 0.89
        // at K = 3072, 0.92 / 1 / 1.05 at 8000, 0.97 / 1 / 1.19 at 25000; v8 m2 0.82 / 1 and v4 m1 0.86 / 1 from 7000 on.  769 to 1024: 1.06 to 1.20,
        // 0.98 to 1.04 and 1.00 to 1.04.)
        if (rows == 128 && blocks(64) > 512 && blocks(64) <= 768 && staged_batch(d, 128, nkt * kSlots * d->vec_len)) rows = 64;
    } else if (d->batch <= 8) {
        if (least == 32 && blocks(32) <= 256 && (d->vec_len == 4 ? codes / 2 : codes) <= 10000000) rows = 32;
        else if (blocks(64) <= 256) rows = 64;
    } else {
        const long long low = d->batch <= 16 ? 8500000 : 4300000;
        if (least == 32 && blocks(32) <= (d->batch <= 16 ? 192 : 256) && codes <= low) rows = 32;
        else if (least <= 64 && !short_groups(d) && blocks(64) <= 256 && (codes <= 8500000 || (d->batch <= 16 && codes <= 16000000 && blocks(64) >= 96))) rows = 64;
    }
    // K ranges.  Up to 4 batch rows: powers of two (others meet through the ticket, 1 us more than two or four pairwise:
    // three ranges are 10 % slower than two or four at any K), up to 256 workgroups, as long as a range is worth its
    // exchange.  One / two ranges break even at K = 4400 (time ratio 0.83 to 0.87 up to 2500, 0.94 at 3500, 1.05 at 6500, 1.2
    // at 14000), two / four at 6000 (0.87 up to 2000, 0.97 at 4500, 1.06 at 7500, 1.12 at 14000), four / eight at 10000 (0.91 up to 9000, 1.09 at
    // 14000, 1.12 from 18000), for 16 to 128 blocks and all formats alike.  More rows: 256 workgroups as long as every
    // wavefront keeps a step (4096^2 at batch 8: two ranges 6.5, one 6.8; 2048^2: two 5.6, four, with half of the
    // wavefronts idle, 6.2).
    const int nb = (int)blocks(rows);
    auto even = [&](int n) { return ceil_div(nkt, ceil_div(nkt, n)) == n; };       // cuts into n ranges, none empty
    // no more workspace than the fields of the Psumbook kernels ask for
    const long long room = (long long)p->k_splits * (d->batch < kBatchPerLaunch ? d->batch : kBatchPerLaunch) / d->batch;
    int splits;
    if (d->batch <= 4) {
        splits = 1;
        while (2 * splits * nb <= 256 && d->in_features >= 2 * splits * (splits == 1 ? 2304 : splits == 2 ? 1792 : 1536)) splits *= 2;
        while (splits > 1 && (splits > room || splits > nkt || !even(splits))) splits /= 2;
    } else {
        splits = 256 / nb;
        const int most = nkt * (d->vec_len == 4 ? 1 : 2) / 8;
        if (splits > most) splits = most;
    }
    if (splits > room) splits = (int)room;
    if (splits > nkt) splits = nkt;
    if (splits < 1) splits = 1;
    // 5 rows and more of the staged kernel's formats: another height or number of ranges where the costs say that it is worth 3 %.  Against the
    // rules alone that is 0.4 % in the mean at 5 to 8 rows, 2 % at 9 to 16, 5 % at 17 to 32 and 4 % above, up to a factor of 2.9; 0.8, 0.6, 1.7 and 2 % of the
    // sizes lose 3 % or more by it (the costs are 9 % off either way).  Two rounds of 128-row blocks and three of 64 rows
    // tie (v8 m2, 5 to 8 rows, 1200 sizes with K from 8192 on, time of 64 / of 128 rows: 1.003 in regions of 3 ms, 0.94 to 1.05; 1.014 in short ones).
    if (d->batch > 4 && staged_format(d)) {
        // v8 m1 without group scales, 17 rows and more: 128-row blocks take 32 rows there and lower ones 16, so these win (0.5 to 0.85 of the time) up to 128
        // tiles of 128 x 32 and lose beyond (1.3 at K = 1000, 1.1 at 3000, 1.03 to 1.08 from 4096 on), whatever K is
        const bool tall = d->vec_len == 8 && d->num_codebooks == 1 && d->group_size < 0 && d->batch > 16 && blocks(128) > 128;
        const int most = nkt * (d->vec_len == 4 ? 1 : 2) / 8;
        float least_cost = 0.97f * batch_cost(d, rows, splits);
        for (int r = tall ? 128 : least; r <= 128; r *= 2)
            for (int n : {1, 2, 3, 4, 6, 8}) {
                const long long workgroups = (long long)n * ceil_div(d->out_features, r) * ceil_div(d->batch, batch_rows(d, r, n));
                if (n > 1 && (workgroups > 256 || n > most || n > room || n > nkt)) break;
                const float cost = batch_cost(d, r, n);
                if (cost >= least_cost) continue;
                least_cost = cost;
                rows = r;
                splits = n;
            }
    }
    p->centroid_rows = rows;
    p->centroid_splits = splits;
    raise_to_staged(d, p);
}

int make_geometry(const codegemm_desc* d, const codegemm_plan* plan, Geometry* g, const codegemm_plan* launch_plan)
{
    int st = validate_desc(d);
    if (st) return st;
    codegemm_plan local;
    if (!plan) {
        choose_plan(d, &local);
        plan = &local;
    }
    st = validate_plan(d, plan);
    if (st) return st;
    codegemm_plan fitted = launch_plan ? *launch_plan : *plan;
    resolve_centroid(d, d->out_features, &fitted);
    plan = &fitted;
    // larger batches run as several launches of the Psumbook kernels, as one of the centroid kernels
    g->B = (d->batch < kBatchPerLaunch || plan->centroid_rows) ? d->batch : kBatchPerLaunch;
    g->K = d->in_features;
    g->N = d->out_features;
    g->v = d->vec_len;
    g->m = d->num_codebooks;
    g->J = g->K / g->v;
    g->NW = plan->waves;
    g->NB = plan->build_waves;
    g->RPL = plan->row_words;
    g->BG = plan->batch_group;
    g->psum_fp16 = plan->psum_dtype == CODEGEMM_PSUM_FP16;
    g->NGR = ceil_div(g->N, kGranuleRows);
    g->RB = plan->centroid_rows;
    if (g->RB) g->BG = centroid_batch(d, g->RB);              // batch rows of a workgroup of the centroid kernel
    // rows per workgroup: 16 per wavefront and row word (32 in the batched kernel)
    g->NBLK = ceil_div(g->NGR * kGranuleRows, g->RPL * (g->NW - g->NB) * (g->BG == 4 ? 32 : 16));
    if (g->RB) g->NBLK = ceil_div(g->N, g->RB);
    g->NKT = ceil_div(g->J, kSlots);
    auto ranges = [&](int want) {               // no empty K range
        const int nks = want < g->NKT ? want : g->NKT;
        return ceil_div(g->NKT, ceil_div(g->NKT, nks));
    };
    g->NKS = g->WKS = ranges(plan->k_splits);
    if (g->RB) {                                // within the workspace of the Psumbook kernel of the same plan
        g->NKS = ranges(plan->centroid_splits);
        const int room = kBatchPerLaunch * g->WKS / g->B;
        if (g->B > kBatchPerLaunch && g->NKS > room) g->NKS = ranges(room > 0 ? room : 1);
    }
    g->KPW = ceil_div(g->NKT, g->NKS);
    g->staged = false;
    if (g->RB) g->BG = batch_rows(d, g->RB, g->NKS, &g->staged);
    // The prompt kernel's workgroups take 1024 rows of W and 64 (with group scales 32) batch rows, or half of the rows and twice the batch rows,
    // and all of K: worth it once they are enough to fill the chip.  fp32 output needs shorter sums than it has (8192^2 v8 m1 g128 batch 512: 2.9e-7
    // of 64 bits, tiles of the centroid kernel 0.95e-7, Psumbook kernels 1.24e-7; 141, 156 and 493 us).
    g->prompt = g->RB && g->B > kBatchPerLaunch && g->v < 16 && !(d->flags & CODEGEMM_FLAG_Y_FP32) &&
                (long long)ceil_div(g->NGR, 8) * ceil_div(g->B, 16 * prompt_tiles(g->m, g->v, d->group_size > 0)) >= 128;
    if (g->prompt) g->NKS = 1;
    // Two wavefronts to a granule make tiles of 512 x 64 of those of 1024 x 32 and take 0.92 of their time (1500 random sizes, 1 to 6
    // rounds of 256 workgroups), but where they are too many for as few rounds (28672 rows, 257 to 288 batch rows: 280 and 252): the
    // other way round is then 1.4 to 1.7 times as fast.
    auto rounds = [&](int granules, int rows) { return ((long long)ceil_div(g->NGR, granules) * ceil_div(g->B, rows) + 255) / 256; };
    g->half = g->prompt && g->v == 4 && g->m == 1 && d->group_size > 0 && 12 * rounds(4, 64) <= 13 * rounds(8, 32);
    g->NG = ceil_div(g->B, g->BG);
    g->Npad = g->NGR * kGranuleRows;
    if (counter_stride(*g) == 0) return CODEGEMM_UNSUPPORTED;   // > 16384 row blocks x batch groups with several K ranges
    g->y_fp32 = (d->flags & CODEGEMM_FLAG_Y_FP32) != 0;
    g->g = d->group_size;
    g->GPU = 0;
    g->gshift = 0;
    if (g->g > 0) {
        const int ratio = g->g / g->v;                 // sub-vectors per group, a power of two
        g->GPU = ratio >= kSlots ? 1 : kSlots / ratio;
        while ((1 << g->gshift) < ratio && g->gshift < 5) ++g->gshift;
    }
    return CODEGEMM_OK;
}

// Geometry of the members of a group under one plan, and the geometry of the whole launch (row
// blocks summed).  The plan has to suit every member, and a launch takes at most kBatchPerLaunch rows.
int group_geometry(const codegemm_desc* desc, const codegemm_plan* plan, const int32_t* out_features,
                   int count, Geometry* members, Geometry* whole)
{
    if (!desc || !out_features) return CODEGEMM_INVALID_ARG;
    if (count < 1 || count > kMaxGroup) return CODEGEMM_INVALID_ARG;
    if (desc->batch > kBatchPerLaunch) return CODEGEMM_UNSUPPORTED;
    codegemm_plan of_sum;
    if (!plan) {   // the default plan of one layer of the summed height, for every member
        const int st = codegemm_default_plan(desc, &of_sum);
        if (st) return st;
        plan = &of_sum;
    }
    long long total = 0;
    for (int i = 0; i < count; ++i) total += out_features[i];
    codegemm_plan fitted = *plan;                      // to the whole launch, so that all members run the same kernel;
                                                       // what is validated is the plan as given: fitting mends invalid fields
    resolve_centroid(desc, total, &fitted);
    for (int i = 0; i < count; ++i) {
        codegemm_desc d = *desc;
        d.out_features = out_features[i];
        const int st = make_geometry(&d, plan, &members[i], &fitted);
        if (st) return st;
    }
    if (total != desc->out_features) return CODEGEMM_INVALID_ARG;
    *whole = members[0];
    whole->N = (int)total;
    whole->NBLK = 0; whole->NGR = 0; whole->Npad = 0;
    for (int i = 0; i < count; ++i) {
        whole->NBLK += members[i].NBLK;
        whole->NGR += members[i].NGR;
        whole->Npad += members[i].Npad;
    }
    if (whole->NBLK > 65535 || counter_stride(*whole) == 0) return CODEGEMM_UNSUPPORTED;
    return CODEGEMM_OK;
}

size_t workspace_counter_bytes(const Geometry&)
{
    return (size_t)kCounterAreaWords * sizeof(uint32_t) + kPairAreaBytes;
}

size_t workspace_need(const Geometry& g)
{
    const size_t floats = (size_t)(g.B < kBatchPerLaunch ? g.B : kBatchPerLaunch) * g.WKS * g.Npad;
    return workspace_counter_bytes(g) + floats * sizeof(float);
}

size_t pair_words(const Geometry& g)
{
    // Measured per level: one add that returns, on every output of the launch at once, takes 0.8-0.9 us, the ticket
    // protocol 1.9 us whatever the number of ranges: two ranges gain 0.95 us, four 0.2 us, eight lose 0.35 us.
    // The batched kernel, with four times the outputs per workgroup, takes it for two ranges only (8192->28672, batch 8:
    // 54.1 -> 53.1 us).  The centroid kernels take it for four as well, at 4 rows too, where a workgroup has no more outputs than the
    // gather kernel's (ticket / pairs: 28672->8192 v8 m2 g128, 4 rows 21.6 / 20.9; 14336->2048 v8 m2, 2 rows 6.08 / 5.93; 33 sizes
    // at 2 to 4 rows 1.011 to 0.969, 0.991 in the mean).
    const bool batched = g.RB == 0 && g.BG == 4;
    if (g.NKS != 2 && (g.NKS != 4 || batched)) return 0;
    return (size_t)g.B * (g.NKS - 1) * g.Npad;
}

int counter_stride(const Geometry& g)
{
    if (g.NKS == 1) return kCounterStride;             // no counter is touched
    const long long blocks = (long long)g.NG * g.NBLK;
    int stride = kCounterStride;
    while (stride > 1 && blocks * stride > kCounterAreaWords) stride /= 2;
    return blocks * stride <= kCounterAreaWords ? stride : 0;
}

}  // namespace cg

using namespace cg;

extern "C" int codegemm_default_plan(const codegemm_desc* desc, codegemm_plan* plan)
{
    if (!plan) return CODEGEMM_INVALID_ARG;
    int st = validate_desc(desc);
    if (st) return st;
    choose_plan(desc, plan);
    return validate_plan(desc, plan);
}

extern "C" size_t codegemm_workspace_bytes(const codegemm_desc* desc, const codegemm_plan* plan)
{
    Geometry g;
    if (make_geometry(desc, plan, &g)) return 0;
    size_t bytes = workspace_need(g);
    if (desc->batch > kBatchPerLaunch && desc->batch % kBatchPerLaunch && !g.RB) {
        // the last launch of a large batch has fewer rows and, under the default plan, other K ranges
        codegemm_desc tail = *desc;
        tail.batch = desc->batch % kBatchPerLaunch;
        if (make_geometry(&tail, plan, &g)) return 0;
        const size_t b2 = workspace_need(g);
        if (b2 > bytes) bytes = b2;
    }
    return bytes;
}

extern "C" size_t codegemm_packed_codes_bytes(const codegemm_desc* desc, const codegemm_plan* plan)
{
    Geometry g;
    if (make_geometry(desc, plan, &g)) return 0;
    return (size_t)g.NGR * g.NKT * kGranuleRows * kSlots * g.m;
}

extern "C" size_t codegemm_packed_scales_bytes(const codegemm_desc* desc)
{
    Geometry g;
    if (make_geometry(desc, nullptr, &g) || g.g <= 0) return 0;
    return (size_t)g.NGR * g.NKT * g.GPU * 256;
}

extern "C" const char* codegemm_status_string(int status)
{
    switch (status) {
        case CODEGEMM_OK: return "ok";
        case CODEGEMM_INVALID_ARG: return "invalid argument";
        case CODEGEMM_UNSUPPORTED: return "unsupported format, batch or plan";
        case CODEGEMM_WORKSPACE_TOO_SMALL: return "workspace too small";
        case CODEGEMM_LAUNCH_FAILED: return "HIP launch failed";
        default: return "unknown status";
    }
}
