// The hot path for batches without a Psumbook: centroid vectors go straight from LDS into the
// matrix cores.  Included by gemm_centroid_m1.hip .. gemm_centroid_m4.hip.
//
// A Psumbook costs 4 bytes of LDS per batch row and code to gather and has to be rebuilt (LDS
// writes, the slow direction) for every 32 sub-vectors of every row block; a centroid costs 2 v
// bytes per code whatever the batch, its table never changes, and v_mfma_f32_16x16x32_f16 takes
// 16 rows x 32 weights of it per instruction.  From two batch rows on that is the cheaper side.
// W is still never formed: each codebook's centroids are multiplied with x on their own (exact
// fp16 products, fp32 accumulation), and scales are applied to fp32 sums.
//
// Mapping onto the packed code layout (no re-ordering).  In v_mfma_f32_16x16x32_f16 lane l of a
// wavefront is column i = l % 16 of the weight operand and slice q = l / 16 of the contraction.
// The columns are row octets of a granule: MFMA u takes row u of every octet, so the 8 rows x 2
// codebooks of one packed 16-byte entry feed 16 MFMAs and no lane needs another lane's codes.
// The other operand is x itself, batch rows along its 16 columns.
// With 8 or 4 batch rows the 16 columns are 8 x 2 or 4 x 4 (batch row, sub-vector), and the
// weight operand's are 8 x 2 or 4 x 4 (octet, sub-vector): only the result elements where the two
// sub-vectors agree mean anything, and they are picked and added over the SB = 2 or 4 lanes at the
// end.  That costs nothing (an instruction takes in 512 weights either way) and puts neighbouring
// lanes on neighbouring entries: with one octet per lane the loads of a quad of lanes fall into
// four cache lines and take 64 clocks instead of 16.  For more than 8 batch rows (SB = 1) pairs of
// loads are made with pairs of lanes along contiguous memory and exchanged in registers.
//
// LDS table: rows of 256 bytes, one per code, each centroid repeated in several columns so that
// the 16 lanes of one LDS cycle read 16 different 16-byte columns whatever the codes are; planes
// of 64 KB.  The byte address (plane << 16) | (code << 8) | column is one byte-permute, as in the
// other kernels.  Two codebooks share the rows of a plane with 8 columns each: lanes 8..15 of a
// row of lanes take the two in the opposite order (their sums do not care), so that at any time
// half of the lanes read one half of the row; four codebooks of 32-byte vectors do the same with
// 4 columns and quads of lanes.
// Measured (random codes, ns per 64-lane read and compute unit): 16 columns of 16 bytes 2.1, 8
// columns 3.5, 4 columns 7, no copies 26; with the MFMA that consumes it 3.1-3.6, 3.9-4.5, 7.4, 26.
//
// The KW wavefronts of a workgroup take consecutive slices of the workgroup's K range for the
// same rows, and their sums meet in LDS: a matrix needs K ranges on different workgroups (and
// the exchange through the workspace) only when N / rows does not fill the chip.
#pragma once

#include "gemm_impl.h"

namespace cg {

typedef __attribute__((address_space(3))) half8_t lds_half8;
typedef __attribute__((address_space(3))) half4_t lds_half4;
typedef __attribute__((address_space(3))) float4_t lds_f4;

template <int M, int V>
struct CentroidTable {
    static constexpr int kEntry = V == 4 ? 8 : 16;                      // bytes one lookup reads
    static constexpr int kHalves = V == 16 ? 2 : 1;                     // lookups per centroid (a plane, or set of planes, each)
    static constexpr int kPlanesPerHalf = V == 16 ? 1 : (M + 1) / 2;
    static constexpr int kBytes = kHalves * kPlanesPerHalf * 65536;
    // Lanes that differ in these bits of i take the codebooks of a plane in another order: codebook k of
    // the program is codebook k ^ order(i) of the lane.
    static constexpr int kOrderBits = (V == 4 || M == 1) ? 0 : (V == 16 && M == 4) ? 2 : 1;
    __host__ __device__ static constexpr int plane(int c, int h) { return V == 16 ? h : c / 2; }
    // region of codebook c in the rows of its plane
    __host__ __device__ static constexpr int region(int c)
    {
        return V == 16 ? (M <= 2 ? (c % 2) * 128 : c * 64) : (c % 2) * 128;
    }
    __host__ __device__ static constexpr int columns(int c)
    {
        const bool alone = c == M - 1 && (M & 1);                       // the last of an odd number has no partner
        const int bytes = V == 16 ? (M == 1 ? 256 : M == 2 ? 128 : alone ? 128 : 64) : alone ? 256 : 128;
        return bytes / kEntry;
    }
};

// 2 x 2 transpose of dwords between two registers and the two lanes of each pair.
__device__ __forceinline__ void pair_transpose(uint32_t& a, uint32_t& b, bool odd)
{
    auto swap1 = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xb1, 0xf, 0xf, true); };   // l <-> l ^ 1
    const uint32_t from_a = swap1(a), from_b = swap1(b);                // before the selects: all lanes take part
    const uint32_t na = odd ? from_b : a, nb = odd ? b : from_a;
    a = na;
    b = nb;
}

// Exchanges two registers' contents between lanes 16 apart: a keeps its rows of lanes 0 and 2 and gets b's there as rows
// 1 and 3, b gets a's rows 1 and 3 as rows 0 and 2.
__device__ __forceinline__ void row_exchange(uint32_t& a, uint32_t& b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}

// Row scale of the output rows of this thread (all of them are row tid % RB of the block), requested in front of the sums over the wavefronts: asked for
// behind them it is the one load that a call still waits for (0.3 to 0.7 us).
template <int RB>
__device__ __forceinline__ uint32_t row_scale_bits(const Member& mm, int tid, int blk)
{
    const int nn = blk * RB + tid % RB;
    return reinterpret_cast<const uint16_t*>(mm.scales)[nn < mm.N ? nn : 0];
}

// Sums over the SLICES partials that the wavefronts have left in LDS, [slice][batch row][RB + 4] (the pad spreads the batch rows over the
// banks), and the end of the workgroup's work.  Each thread adds up the outputs that it then stores; all tiles of batch rows
// together: one barrier in front and one behind, where a tile at a time with its totals in LDS took 0.5 (8 rows) to 1.7 us (16 rows in
// 32-row blocks) of a call.
template <int THREADS, int BT, int RB, int SLICES, bool TERNARY = false>
struct SliceSums {
    static constexpr int kStride = RB + 4;
    static constexpr size_t kBytes = (size_t)SLICES * BT * kStride * sizeof(float);
    static constexpr size_t kLds = kBytes + 64;        // .. and the ticket's flag
    static __device__ __forceinline__ void finish(const GemmParams& p, const Member& mm, float* parts, uint32_t scale_bits, int tid, int blk, int ks, int b0)
    {
        finish_block<THREADS, BT, RB, SLICES, TERNARY>(p, mm, parts, reinterpret_cast<uint32_t*>(reinterpret_cast<unsigned char*>(parts) + kBytes), tid, blk, ks, b0, scale_bits);
    }
};

// The one pass costs some instances of gemm_centroid_kernel, whose registers are all taken, values of the loop that go to scratch.  (Percent of a call's time, on
// random sizes with 9 batch rows and more, against sums a tile at a time; lowest and highest in brackets.)
//  * fp32 output, v8 m1 with group scales, 32-row blocks (27 spills for 11): 2 to 4 % more (-5 to 14).  It keeps sums a tile at a time.
//  * 128-row blocks of fp16 output v16 m4 (19 for 18) 5 % more (0 to 12), of v16 m3 with groups that hold a step and of fp32 output v4 m2 with group
//    scales 0 % (-4 to 7).  What outputs beyond the batch do not add, written as a conditional expression in place of a branch, gives them another
//    assignment of registers: 1 to 3 % less, 2 % less and 2 % less (none more than 1 % more).  Other instances spill more by it (fp32 output v8 m4 and
//    v4 m2, v8 m4 with group scales: 1 to 13 % more time).
__host__ __device__ constexpr bool sums_tiled(int m, int v, int sb, int nt, int gs) { return m == 1 && v == 8 && sb == 4 && nt == 4 && gs == 4; }
__host__ __device__ constexpr bool sums_ternary(int m, int v, int sb, int gs)
{
    return sb == 1 && ((m == 4 && v == 16 && gs == 0) || (m == 3 && v == 16 && gs == 1) || (m == 2 && v == 4 && gs == 4));
}

// SB: sub-vectors along the columns of the operands (16 / SB octets per wavefront, 16 / SB batch rows per tile).
// NT: tiles of batch rows.  RW x KW wavefronts: RW blocks of 128 / SB rows, KW slices of K.  D: steps in the load
// ring.  GS: 0 one scale per row; 1 group scales, a step (16 chunks) lies in one group; 2 groups of 4 or 8 chunks (a
// chunk is a sub-vector, two for v = 4): every MFMA then contracts over 4 neighbouring chunks instead of chunks 4 apart,
// and sums are scaled after every round; 3 and 4 fp32 output, short chains of sums, with one scale per row and with group
// scales (chunks as for 2).  ONE (SB = 4): one batch row, for which the result elements are arranged so that a lane has
// one that means something instead of one of four.
//
// GS = 3 and 4.  Every MFMA on an accumulator rounds it, and a wavefront's share of K is hundreds of them in a row: up to
// four times the error of the Psumbook kernels against 64 bits, which is lost in the rounding of fp16 output (2.1e-4) but
// not here.  Measured on random operands (relative rms, 1e-7): an MFMA of 32 products 0.44, two on one accumulator 0.57,
// four 0.76; the Psumbook's 8 products 0.31.  The Psumbook kernels spread K over 32 lanes (16 in the batched kernel) and
// their K ranges, more than the sub-vectors, slices and ranges here, so chains have to be shorter and sums have a second
// level.  A result tile takes two MFMAs (three codebooks at 5 to 8 rows: three; GS = 4: one, the tiles of a round being added
// before they are scaled; two above 8 batch rows and the whole round for v = 4, whose Psumbook adds twice as often) and is then added to sums of its own, which
// go to totals after 8 to 16 additions.  Error against that of the Psumbook plan of the same call, fp32 output, geometric
// mean over some hundred random sizes per format and power of two of K: at most 1.00, 0.4 to 0.95 from K = 4096 on
// (8192^2, batch 512, 1e-7: v8 m2 1.06 against 1.32, v8 m1 g128 0.95 against 1.24, v8 m2 g32 1.01 against 1.60).  It costs
// up to 10 % against chains of four (8192^2 v8 m2 batch 4 11.2 -> 11.1 us, 4120->11111 v8 m3 batch 5 13.60 -> 13.80).
template <int M, int V, int SB, int NT, int RW, int KW, int D, int GS, bool ONE>
__global__ void __launch_bounds__(RW * KW * 64) gemm_centroid_kernel(CG_HEAD_PARAMS, const GemmParams pk)
{
    const GemmParams p = with_head(pk, hx, hpacked, hcodebooks, hgscales, hK, hNKT, hKPW, hB, hNGR, hmisc);
    typedef CentroidTable<M, V> T;
    constexpr int THREADS = RW * KW * kWave;
    constexpr int OCT = 16 / SB;                       // octets of a wavefront
    constexpr int RB = 8 * OCT * RW;                   // rows of the workgroup
    constexpr int BPT = ONE ? 1 : 16 / SB;             // batch rows per tile
    static_assert(!ONE || (SB == 4 && NT == 1), "one batch row");
    constexpr int BT = BPT * NT;                       // batch rows of the workgroup
    constexpr int SPU = V == 4 ? 1 : 2;                // steps per unit of 32 sub-vectors
    constexpr int R = 4 / SB;                          // rounds per step: 4 SB chunks of 16 bytes of x (v = 16: 32) each
    constexpr int HALVES = T::kHalves;                 // operands of 8 elements per chunk
    constexpr int NSB = R * HALVES * M;                // (round, half, codebook) per step: 8 lookups and 8 NT MFMAs each
    constexpr int PW = V == 4 ? 8 : 4;                 // dwords per lane and round of a part with two codebooks
    constexpr int WR = PW / 2 * M;                     // .. of all parts
    constexpr int CHUNK = V == 16 ? 16 : 8;            // elements of x per chunk
    constexpr int kUnitBytes = kGranuleRows * kSlots * M;
    constexpr bool SCALED = GS == 1 || GS == 2 || GS == 4;
    constexpr bool NEAR = GS == 2 || GS == 4;          // an MFMA contracts over 4 neighbouring chunks
    constexpr bool SHORT = GS >= 3;
    constexpr int ROUND = NEAR ? M * HALVES : NSB;     // (half, codebook) of a round, which share a scale
    // MFMAs in a row on a result tile, before it is added to the sums; the tile starts and ends with them
    constexpr int LINK = GS == 3 ? (M == 3 && SB == 2 ? 3 : 2) : GS == 4 && V > 4 ? (SB > 1 ? 1 : 2) : ROUND;
    auto starts = [](int k) constexpr -> bool { return GS != 0 && k % ROUND % LINK == 0; };
    auto ends = [](int k) constexpr -> bool { return GS != 0 && (k % ROUND % LINK == LINK - 1 || k % ROUND == ROUND - 1); };
    constexpr bool PARTS = GS == 4 && LINK == 1 && ROUND > 1;       // the tiles of a round are added before they are scaled
    // SHORT: the sums are moved to the totals after 8 to 12 additions (SB = 2, whose error leaves room for it: 12 to 16):
    // every step, or every few turns of the ring
    constexpr int ADDS = (NSB / ROUND) * (PARTS ? 1 : (ROUND + LINK - 1) / LINK);            // per step
    constexpr int AIM = SB == 2 ? 16 : 8;
    constexpr int TURNS = ADDS >= AIM ? 0 : D * ADDS >= AIM ? 1 : D * ADDS >= AIM / 2 ? 2 : 4;
    constexpr int kOutOfRange = 0x7ffffff0;
    constexpr uint32_t kRsrcFlags = 0x00020000u;
    constexpr bool TILED = sums_tiled(M, V, SB, NT, GS);
    // The row scale is asked for behind the loop, in front of the wavefronts' sums: with the first codes it held a register through the loop and
    // made calls 1 to 3 % longer.  Here that register happens to leave the loop fewer spills (7 for 12): 0.88 of the time, 9 batch rows and more.
    constexpr bool EARLY = GS == 3 && V == 4 && M == 2 && SB == 1;
    static_assert((KW & (KW - 1)) == 0, "slices are added in pairs");
    static_assert(THREADS == 512, "a pass over the table's entries is one codebook (v = 16) or two");
    static_assert(RB <= kGranuleRows, "rows of a workgroup lie in one granule");

    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rw = wave % RW, kw = wave / RW;
    const int ks = blockIdx.x;
    const Member mm = member_of(p, blockIdx.y);
    const int blk = blockIdx.y - mm.blk0;
    const int b0 = blockIdx.z * BT;
    const int kt0 = ks * p.KPW;
    const int nq = min(p.KPW, p.NKT - kt0);
    const int q = lane >> 4;
    // columns of the operands: octet (batch row) and sub-vector; with SB = 1 the loads pair up lanes as with SB = 2
    // and the exchange leaves octet (batch row) lane % 16 to the lane
    constexpr int LS = SB == 1 ? 2 : SB;
    const int ls = lane & (LS - 1), lo = (lane & 15) / LS;
    const int col_o = (lane & 15) / SB;                // octet of this lane's column
    const bool odd = lane & 1;
    // Chunk of load j of a step: the lane's part and the load's (chunk_at(j)).  SB = 1: loads 2 i and 2 i + 1 take the same
    // chunk of two octets (batch rows), exchanged afterwards; GS = 2 moves chunk bits between lanes 16 apart as well.
    auto lane_chunk = [&](int sv) -> int {             // sv: the lane's place along contiguous memory
        if constexpr (NEAR) return SB == 1 ? 4 * (q & 1) + 2 * (q >> 1) + sv : 4 * sv + q;
        else return 4 * q + sv;
    };
    auto chunk_at = [](int j) -> int {
        if constexpr (SB == 1) return (NEAR ? 8 : 2) * (j / 2);
        else return (NEAR ? 4 * SB : SB) * j;
    };

    // Table entries of this thread, requested first: everything waits for them.  A pass takes THREADS entries, whole codebooks with as many
    // columns each; where fewer are left, several threads share the columns of one.
    constexpr int ENTRIES = M * kCentroids * T::kHalves;                // to replicate
    constexpr int EPT = (ENTRIES + THREADS - 1) / THREADS;              // passes
    auto sharing = [](int k) constexpr -> int { return ENTRIES - k * THREADS < THREADS ? THREADS / (ENTRIES - k * THREADS) : 1; };
    typedef typename Frag<V == 4 ? 4 : 16>::type entry_t;               // 8 or 16 bytes
    entry_t fill[EPT];
#pragma unroll
    for (int k = 0; k < EPT; ++k)
        fill[k] = reinterpret_cast<const entry_t*>(mm.codebooks)[k * THREADS + tid / sharing(k)];      // entry e = (codebook, centroid, half) in memory order

    // This wavefront's steps [s_beg, s_end) of the workgroup's K range.
    const int total = nq * SPU;
    const int s_beg = total * kw / KW, s_end = total * (kw + 1) / KW;

    // x: round j of a step, chunk lane_chunk + chunk_at(j) of the step's 16 (SB = 1: loads 2 i and 2 i + 1 of batch rows
    // 2 lo and 2 lo + 1; after the exchange register j is chunk 4 q + j, or 4 j + q with GS = 2, of row lane % 16)
    const __amdgpu_buffer_rsrc_t x_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<_Float16*>(p.x + (size_t)b0 * p.K), 0, min(p.B - b0, BT) * p.K * 2, kRsrcFlags);
    const int xb = ONE ? lane & 3 : lo, xs = ONE ? (lane >> 2) & 3 : ls;           // ONE: batch row innermost
    const int x_el0 = kt0 * kSlots * V + lane_chunk(xs) * CHUNK;
    const int x_off = ((SB == 1 ? 2 * xb : xb) * p.K + x_el0) * 2;
    auto load_x = [&](half8_t (&dst)[NT][R][HALVES], int s) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int el = s * (16 * CHUNK) + chunk_at(j) * CHUNK;
            const int at = (s < s_end && x_el0 + el < p.K) ? el * 2 + (SB == 1 ? (j % 2) * p.K * 2 : 0) : kOutOfRange;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int h = 0; h < HALVES; ++h)
                    dst[nt][j][h] = __builtin_bit_cast(half8_t, __builtin_amdgcn_raw_buffer_load_b128(x_rsrc, x_off + nt * BPT * 2 * p.K + at + 16 * h, 0, 0));
        }
    };
    auto turn_x = [&](half8_t (&xv)[NT][R][HALVES], int s) {
        if constexpr (V == 4) {                        // an odd number of sub-vectors: the chunk may reach past the end of the row
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const bool past = x_el0 + s * (16 * CHUNK) + chunk_at(j) * CHUNK + 4 >= p.K;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    u32x4_t t = __builtin_bit_cast(u32x4_t, xv[nt][j][0]);
                    t.z = past ? 0u : t.z;
                    t.w = past ? 0u : t.w;
                    xv[nt][j][0] = __builtin_bit_cast(half8_t, t);
                }
            }
        }
        if constexpr (SB == 1) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int j = 0; j < R; j += 2)
#pragma unroll
                    for (int h = 0; h < HALVES; ++h) {
                        u32x4_t a = __builtin_bit_cast(u32x4_t, xv[nt][j][h]), b = __builtin_bit_cast(u32x4_t, xv[nt][j + 1][h]);
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            uint32_t ak = a[k], bk = b[k];
                            pair_transpose(ak, bk, odd);
                            if constexpr (NEAR) row_exchange(ak, bk);
                            a[k] = ak;
                            b[k] = bk;
                        }
                        xv[nt][j][h] = __builtin_bit_cast(half8_t, a);
                        xv[nt][j + 1][h] = __builtin_bit_cast(half8_t, b);
                    }
        }
    };
    // Codes of round j: octet lo, sub-vector 16 (s % 2) + chunk (v = 4: sub-vectors 2 chunk and 2 chunk + 1), pairs of
    // loads for SB = 1 as above.
    const int row0 = blk * RB + rw * (8 * OCT);
    const int gr = row0 / kGranuleRows;
    const int oct0 = (row0 % kGranuleRows) / kRowsPerLane;
    const uint8_t* cbase = mm.packed + ((size_t)min(gr, mm.NGR - 1) * p.NKT + kt0) * kUnitBytes;
    const __amdgpu_buffer_rsrc_t c_rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(cbase), 0, gr < mm.NGR ? nq * kUnitBytes : 0, kRsrcFlags);
    const int c_ent = (oct0 + (SB == 1 ? 2 * lo : lo)) * kSlots + (V == 4 ? 2 : 1) * lane_chunk(ls);
    auto load_codes = [&](uint32_t (&dst)[R][WR], int s) {
        const int unit = s < s_end ? (s / SPU) * kUnitBytes : kOutOfRange;
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int ent = c_ent + (V == 4 ? 0 : (s % SPU) * 16) + (V == 4 ? 2 : 1) * chunk_at(j) + (SB == 1 ? (j % 2) * kSlots : 0);
#pragma unroll
            for (int part = 0; part < (M + 1) / 2; ++part) {
                uint32_t* w = dst[j] + part * PW;
                if (2 * part + 1 == M) {               // last part of an odd m: 8 bytes per entry
                    if constexpr (V == 4) {
                        const u32x4_t t = __builtin_amdgcn_raw_buffer_load_b128(c_rsrc, unit + part * 8192 + ent * 8, 0, 2);
                        w[0] = t.x; w[1] = t.y; w[2] = t.z; w[3] = t.w;
                    } else {
                        const u32x2_t t = __builtin_amdgcn_raw_buffer_load_b64(c_rsrc, unit + part * 8192 + ent * 8, 0, 2);
                        w[0] = t.x; w[1] = t.y;
                    }
                } else {
#pragma unroll
                    for (int g = 0; g < PW / 4; ++g) {
                        const u32x4_t t = __builtin_amdgcn_raw_buffer_load_b128(c_rsrc, unit + part * 8192 + (ent + g) * 16, 0, 2);
                        w[4 * g] = t.x; w[4 * g + 1] = t.y; w[4 * g + 2] = t.z; w[4 * g + 3] = t.w;
                    }
                }
            }
        }
    };
    // The exchange of SB = 1, then the lane's order of the codebooks that share a plane.
    const int order = T::kOrderBits == 2 ? (lane >> 2) & 3 : T::kOrderBits == 1 ? (lane >> 3) & 1 : 0;
    auto turn_codes = [&](uint32_t (&cw)[R][WR]) {
        if constexpr (SB == 1) {
#pragma unroll
            for (int j = 0; j < R; j += 2)
#pragma unroll
                for (int k = 0; k < WR; ++k) {
                    pair_transpose(cw[j][k], cw[j + 1][k], odd);
                    if constexpr (NEAR) row_exchange(cw[j][k], cw[j + 1][k]);
                }
        }
        if constexpr (T::kOrderBits > 0) {
#pragma unroll
            for (int j = 0; j < R; ++j) {
#pragma unroll
                for (int part = 0; part < M / 2; ++part)
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        uint32_t* w = cw[j] + part * PW;
                        const uint32_t a = w[k], b = w[2 + k];
                        w[k] = (order & 1) ? b : a;
                        w[2 + k] = (order & 1) ? a : b;
                    }
                if constexpr (T::kOrderBits == 2) {
#pragma unroll
                    for (int k = 0; k < PW; ++k) {
                        const uint32_t a = cw[j][k], b = cw[j][PW + k];
                        cw[j][k] = (order & 2) ? b : a;
                        cw[j][PW + k] = (order & 2) ? a : b;
                    }
                }
            }
        }
    };
    // group scales of the lane's octet for the group of step s
    __amdgpu_buffer_rsrc_t s_rsrc;
    if constexpr (SCALED) {
        const uint8_t* base = mm.gscales + ((size_t)min(gr, mm.NGR - 1) * p.NKT + kt0) * p.GPU * 256;
        s_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(base), 0, gr < mm.NGR ? nq * p.GPU * 256 : 0, kRsrcFlags);
    }
    constexpr int SR = NEAR ? R : 1;                // scales per step
    auto load_scales = [&](half8_t (&dst)[SR], int s) {
#pragma unroll
        for (int j = 0; j < SR; ++j) {
            // first sub-vector, in its unit, of the chunks that the lane's column contracts over
            const int chunk = NEAR ? (SB == 1 ? 4 * j : chunk_at(j) + 4 * (lane & (SB - 1))) : 0;
            const int sub = (s % SPU) * 16 + (V == 4 ? 2 : 1) * chunk;
            const int o = s < s_end ? ((s / SPU) * p.GPU + (sub >> p.gshift)) * 256 : kOutOfRange;
            dst[j] = __builtin_bit_cast(half8_t, __builtin_amdgcn_raw_buffer_load_b128(s_rsrc, o + (oct0 + col_o) * 16, 0, 0));
        }
    };

    half8_t xr[D][NT][R][HALVES];
    uint32_t w[D][R][WR];
    half8_t sc[SCALED ? D : 1][SR];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int d = 0; d < D; ++d) {
        load_codes(w[d], s_beg + d);
        load_x(xr[d], s_beg + d);
        if constexpr (SCALED) load_scales(sc[d], s_beg + d);
    }
    uint32_t scale_bits = 0x3c00u;
    if constexpr (EARLY) scale_bits = row_scale_bits<RB>(mm, tid, blk);
    __builtin_amdgcn_sched_barrier(0);

    // replicate the centroids
    const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>((lds_float*)smem);
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
        const int share = sharing(k), e = k * THREADS + tid / share;
        const int h = e % T::kHalves, code = (e / T::kHalves) % kCentroids, c = e / (T::kHalves * kCentroids);
        // columns this thread fills, beginning at another one in every row so that a wavefront's stores spread over the banks
        const int cols = T::columns(k * THREADS / (T::kHalves * kCentroids)), mine = cols / share;
        const int c0 = tid % share * mine + (tid / share & (mine - 1));
        const uint32_t first = lds0 + (uint32_t)(T::plane(c, h) * 65536 + code * 256 + T::region(c) + c0 * T::kEntry);
#pragma unroll
        for (int j = 0; j < mine; ++j) {
            const uint32_t a = first ^ (uint32_t)(j * T::kEntry);
            if constexpr (V == 4) *reinterpret_cast<lds_half4*>(static_cast<uintptr_t>(a)) = fill[k];
            else *reinterpret_cast<lds_half8*>(static_cast<uintptr_t>(a)) = fill[k];
        }
    }

    // Result tiles; with group scales or fp32 output those of one chain, and the (scaled) sums of the elements
    // that mean something beside them.
    float4_t acc[NT][8];
    constexpr int TL = 4 / SB;                         // batch rows of a lane per tile
    float sum[GS ? NT : 1][8][GS ? TL : 1], total_of[SHORT ? NT : 1][8][SHORT ? TL : 1], part[PARTS ? NT : 1][8][PARTS ? TL : 1];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            acc[nt][u] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
            if constexpr (GS) {
#pragma unroll
                for (int t = 0; t < TL; ++t) {
                    sum[nt][u][t] = 0.0f;
                    if constexpr (SHORT) total_of[nt][u][t] = 0.0f;
                }
            }
        }
    // Batch row t of this lane in a result tile, whose row 4 q + e is batch row 4 q + e for SB = 1; batch row 2 q + e / 2,
    // sub-vector e % 2 for SB = 2; batch row q, sub-vector e for SB = 4: the meaningful elements are those of the column's
    // own sub-vector.  ONE: batch row e, sub-vector q, meaningful in the lanes whose column has sub-vector q.
    auto own = [&](const float4_t& r, int t) -> float {
        if constexpr (SB == 1 || ONE) return r[t];
        else if constexpr (SB == 2) return odd ? r[2 * t + 1] : r[2 * t];
        else {
            const float lo2 = odd ? r[1] : r[0], hi2 = odd ? r[3] : r[2];
            return (lane & 2) ? hi2 : lo2;
        }
    };

    // Lookup bases: plane, region and column of codebook k as this lane orders them, per half.
    uint32_t base[M][HALVES];
#pragma unroll
    for (int k = 0; k < M; ++k) {
        const bool alone = k == M - 1 && (M & 1);
        const int c = alone ? k : k ^ order;
        const uint32_t at = lds0 + (uint32_t)((alone ? T::region(k) : T::kOrderBits == 2 ? c * 64 : T::kOrderBits == 1 ? (c % 2) * T::region(1) : T::region(k)) +
                                              (lane & (T::columns(k) - 1)) * T::kEntry);
#pragma unroll
        for (int h = 0; h < HALVES; ++h) base[k][h] = at + (uint32_t)(T::plane(k, h) << 16);
    }
    // Centroid operand of MFMA u in (round, half, codebook) k of a step: row u of the lane's octet.
    auto fetch = [&](const uint32_t (&cw)[R][WR], int k, int u) -> half8_t {
        const int c = k % M, h = (k / M) % HALVES, j = k / (M * HALVES);
        const uint32_t* w = cw[j] + (c / 2) * PW;
        const bool single = 2 * (c / 2) + 1 == M;
        const uint32_t sel = 0x0c020000u | (uint32_t)(4 + u % 4) << 8;
        if constexpr (V == 4) {
            const uint32_t w0 = single ? w[u / 4] : w[2 * (c % 2) + u / 4], w1 = single ? w[2 + u / 4] : w[4 + 2 * (c % 2) + u / 4];
            const half4_t lo4 = *reinterpret_cast<const lds_half4*>(static_cast<uintptr_t>(__builtin_amdgcn_perm(w0, base[c][0], sel)));
            const half4_t hi4 = *reinterpret_cast<const lds_half4*>(static_cast<uintptr_t>(__builtin_amdgcn_perm(w1, base[c][0], sel)));
            return __builtin_shufflevector(lo4, hi4, 0, 1, 2, 3, 4, 5, 6, 7);
        } else {
            const uint32_t w0 = single ? w[u / 4] : w[2 * (c % 2) + u / 4];
            return *reinterpret_cast<const lds_half8*>(static_cast<uintptr_t>(__builtin_amdgcn_perm(w0, base[c][h], sel)));
        }
    };

    auto add_scaled = [&](const half8_t& scales) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float f = (float)scales[u];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int t = 0; t < TL; ++t) {
                    float& x = sum[SCALED ? nt : 0][u][SCALED ? t : 0];
                    x = __builtin_fmaf(f, PARTS ? part[PARTS ? nt : 0][u][PARTS ? t : 0] : own(acc[nt][u], t), x);
                    if constexpr (SHORT) asm volatile("" : "+v"(x));
                }
        }
    };

    auto add_part = [&](bool first) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int t = 0; t < TL; ++t) {
                    float& x = part[PARTS ? nt : 0][u][PARTS ? t : 0];
                    const float r = own(acc[nt][u], t);
                    x = first ? r : x + r;
                    asm volatile("" : "+v"(x));
                }
    };
    auto add_up = [&]() {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int t = 0; t < TL; ++t) {
                    float& x = sum[GS ? nt : 0][u][GS ? t : 0];
                    x += own(acc[nt][u], t);
                    asm volatile("" : "+v"(x));        // here: the compiler would keep the tiles and add them all later
                }
    };

    auto move_up = [&]() {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int t = 0; t < TL; ++t) {
                    total_of[SHORT ? nt : 0][u][SHORT ? t : 0] += sum[GS ? nt : 0][u][GS ? t : 0];
                    sum[GS ? nt : 0][u][GS ? t : 0] = 0.0f;
                }
    };

    __syncthreads();

    // Main loop.  Every MFMA is followed by the lookup that takes its operand's registers, for the same u
    // of the next (round, half, codebook): eight lookups are in flight while the matrix cores work.
    half8_t a[8];
    turn_codes(w[0]);
#pragma unroll
    for (int u = 0; u < 8; ++u) a[u] = fetch(w[0], 0, u);
    int turn = 0;
    for (int s0 = s_beg; s0 < s_end; s0 += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int s = s0 + d;
            turn_codes(w[(d + 1) % D]);
            if (s < s_end) {
                turn_x(xr[d], s);
#pragma unroll
                for (int k = 0; k < NSB; ++k) {
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) {
                            const half8_t xv = xr[d][nt][k / (M * HALVES)][(k / M) % HALVES];
                            acc[nt][u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xv, a[u], starts(k) ? float4_t{} : acc[nt][u], 0, 0, 0);
                        }
                        __builtin_amdgcn_sched_barrier(0);         // the lookup after its operand's last use: no second set of registers
                        a[u] = k + 1 < NSB ? fetch(w[d], k + 1, u) : fetch(w[(d + 1) % D], 0, u);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (ends(k)) {
                        if constexpr (GS == 3) add_up();
                        if constexpr (PARTS) add_part(k % ROUND == 0);
                        if constexpr (SCALED) if (!PARTS || k % ROUND == ROUND - 1) add_scaled(sc[d][NEAR ? k / ROUND : 0]);
                    }
                }
            }
            if constexpr (SHORT && TURNS == 0) move_up();
            load_codes(w[d], s + D);
            load_x(xr[d], s + D);
            if constexpr (SCALED) load_scales(sc[d], s + D);
        }
        if constexpr (SHORT && TURNS > 0) {
            if (++turn % TURNS == 0) move_up();
        }
    }
    if constexpr (SHORT) move_up();

    // Sum over the wavefronts' K slices: partials in LDS (ONE: the four sub-vectors of a slice apart), all tiles of batch rows at once or (TILED) one
    // by one, the totals then behind them as [batch row][RB].
    constexpr int SLICES = ONE ? 4 * KW : KW;
    constexpr int ROWS = TILED ? BPT : BT;
    typedef SliceSums<THREADS, ROWS, RB, SLICES, sums_ternary(M, V, SB, GS)> Sums;
    float* parts = reinterpret_cast<float*>(smem);
    float* totals = parts + SLICES * ROWS * Sums::kStride;
    __syncthreads();                                   // everyone is done with the table
    if constexpr (!SCALED && !EARLY && !TILED) scale_bits = row_scale_bits<RB>(mm, tid, blk);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        if (TILED && nt > 0) __syncthreads();          // the previous tile's partials have been read
#pragma unroll
        for (int t = 0; t < TL; ++t) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                v[u] = SHORT ? total_of[SHORT ? nt : 0][u][SHORT ? t : 0] : GS ? sum[GS ? nt : 0][u][GS ? t : 0] : own(acc[nt][u], t);
                if constexpr (SB >= 2 && !ONE) v[u] = dpp_add<0xb1, 0xf>(v[u]);
                if constexpr (SB == 4 && !ONE) v[u] = dpp_add<0x4e, 0xf>(v[u]);
            }
            const int b = ONE ? 0 : BPT * nt + TL * q + t;
            if (ONE ? (lane & 3) == q : b0 + b < p.B && (lane & (SB - 1)) == 0) {
                float* dst = parts + ((ONE ? kw * 4 + q : kw) * ROWS + b % ROWS) * Sums::kStride + (rw * OCT + col_o) * 8;
                *reinterpret_cast<float4_t*>(dst) = float4_t{v[0], v[1], v[2], v[3]};
                *reinterpret_cast<float4_t*>(dst + 4) = float4_t{v[4], v[5], v[6], v[7]};
            }
        }
        if constexpr (TILED) {
            __syncthreads();
            const int nb = min(p.B - b0 - BPT * nt, BPT);
            for (int o = tid; o < nb * RB; o += THREADS)
                totals[BPT * nt * RB + o] = pairwise_sum<SLICES>(parts + o / RB * Sums::kStride + o % RB, BPT * Sums::kStride);
        }
    }
    if constexpr (TILED) finish_block<THREADS, BT, RB>(p, mm, totals, reinterpret_cast<uint32_t*>(totals + BT * RB), tid, blk, ks, b0);
    else Sums::finish(p, mm, parts, scale_bits, tid, blk, ks, b0);
}

// Steps in the load ring of the kernels with one tile of batch rows: four, but three or two where that is what brings a lane's
// registers down to 128.  One or two codebooks of short vectors take 64 KB of LDS, so in launches of more than 256 workgroups two then share
// a compute unit, and each fills the other's first loads, table and exchange (8192->57344 v8 m2 g128, 4 rows: 134 registers 45.1 us,
// 122 registers 40.4).  Time of four steps / time here, 3800 random sizes: above 256 workgroups 1.05 to 1.24 with a K below 8192, 1.00 to 1.15
// beyond.  It wins with one workgroup on a compute unit too, by some 0.4 us a call (why is not known): 32-row blocks 1.05 to 1.08
// below K = 3072, 0.99 to 1.09 above; 64-row blocks 1.05 to 1.08 and 0.96 to 1.09; 128-row blocks of two codebooks 1.04 to 1.06 and 1.00 to 1.06, of
// one 1.01 and 0.94 to 1.01 (v8 fp32 output with group scales is the format below 0.96; its sums move to the totals once a turn, so that the
// depth has to be the same at any number of workgroups).  5 to 8 rows, v4 m1: 1.07, with group scales 1.14.  Where both depths fit,
// the deeper one wins (8B block, v4 m1 g128, one row: three steps 30.4 us, four 28.8).
__host__ __device__ constexpr int centroid_ring(int m, int v, int sb, int gs, bool one)
{
    const bool shared = v < 16 && m <= 2;              // the table leaves room for a second workgroup
    if (sb == 4) return shared && (m == 2 ? gs == 1 || (gs == 2 && v == 8) : !one && (gs == 4 || (v == 4 && gs == 2))) ? 3 : 4;
    if (shared && m == 1 && v == 4 && gs <= 1) return gs == 1 ? 2 : 3;
    return gs == 2 || gs == 4 ? 3 : 4;
}

template <int M, int V, int SB, int NT, int RW, int KW, int D, int GS, bool ONE = false>
int launch_gemm_centroid_one(const Geometry& g, const GemmParams& p, hipStream_t stream)
{
    auto fn = gemm_centroid_kernel<M, V, SB, NT, RW, KW, D, GS, ONE>;
    constexpr int RB = 128 / SB * RW, BPT = ONE ? 1 : 16 / SB;
    if (g.RB != RB || g.BG != BPT * NT) return CODEGEMM_UNSUPPORTED;
    constexpr bool TILED = sums_tiled(M, V, SB, NT, GS);
    constexpr size_t stage = SliceSums<RW * KW * kWave, TILED ? BPT : BPT * NT, RB, ONE ? 4 * KW : KW>::kLds + (TILED ? BPT * NT * RB * sizeof(float) : 0);
    constexpr size_t table = CentroidTable<M, V>::kBytes;
    constexpr size_t lds = stage > table ? stage : table;
    static_assert(lds <= (size_t)kMaxLds, "LDS");
    int st = set_max_lds(reinterpret_cast<const void*>(fn), lds);
    if (st != CODEGEMM_OK) return st;
    const dim3 grid((unsigned)g.NKS, (unsigned)g.NBLK, (unsigned)g.NG);
    hipLaunchKernelGGL(fn, grid, dim3(RW * KW * kWave), lds, stream, CG_HEAD_ARGS(p), p);
    return hipGetLastError() == hipSuccess ? CODEGEMM_OK : CODEGEMM_LAUNCH_FAILED;
}

template <int M, int V, int GS>
int launch_gemm_centroid_v(const Geometry& g, const GemmParams& p, hipStream_t stream)
{
    // From 5 rows on fp16 output of one or two codebooks has a kernel of its own (gemm_staged_impl.h), but for two shapes that do not fit there
    // and short K
    constexpr bool STAGED = GS <= 2 && ((V == 8 && M <= 2) || (V == 4 && M == 1)), WIDE = V == 8 && M == 1;
    constexpr int D1 = centroid_ring(M, V, 4, GS, true), D4 = centroid_ring(M, V, 4, GS, false), D2 = centroid_ring(M, V, 2, GS, false);
    switch (g.BG) {
        case 1:
            if (g.RB == 128) return launch_gemm_centroid_one<M, V, 4, 1, 4, 2, D1, GS, true>(g, p, stream);
            if (g.RB == 64) return launch_gemm_centroid_one<M, V, 4, 1, 2, 4, D1, GS, true>(g, p, stream);
            return launch_gemm_centroid_one<M, V, 4, 1, 1, 8, D1, GS, true>(g, p, stream);
        case 4:
            if (g.RB == 128) return launch_gemm_centroid_one<M, V, 4, 1, 4, 2, D4, GS>(g, p, stream);
            if (g.RB == 64) return launch_gemm_centroid_one<M, V, 4, 1, 2, 4, D4, GS>(g, p, stream);
            return launch_gemm_centroid_one<M, V, 4, 1, 1, 8, D4, GS>(g, p, stream);
        case 8:
            if constexpr (!STAGED || V == 4 || GS == 0 || (WIDE && GS == 2)) {
                if (g.RB == 128) return launch_gemm_centroid_one<M, V, 2, 1, 2, 4, D2, GS>(g, p, stream);
            }
            if constexpr (!STAGED) {
                if (g.RB == 64) return launch_gemm_centroid_one<M, V, 2, 1, 1, 8, D2, GS>(g, p, stream);
                if constexpr (V < 16) return launch_gemm_centroid_one<M, V, 4, 2, 1, 8, 3, GS>(g, p, stream);
            }
            break;
        case 16:
            if constexpr (!STAGED || WIDE) {
                if (g.RB == 128) return launch_gemm_centroid_one<M, V, 1, 1, 1, 8, 2, GS>(g, p, stream);
            }
            if constexpr (!STAGED && V < 16 && ((GS != 2 && GS != 4) || M == 1)) {
                if (g.RB == 64) return launch_gemm_centroid_one<M, V, 2, 2, 1, 8, 2, GS>(g, p, stream);
            }
            if constexpr (!STAGED && V < 16 && (GS == 0 || M == 1)) {
                if (g.RB == 32) return launch_gemm_centroid_one<M, V, 4, 4, 1, 8, 2, GS>(g, p, stream);
            }
            break;
        case 32:
            if constexpr (GS == 0 && WIDE) return launch_gemm_centroid_one<M, V, 1, 2, 1, 8, 2, GS>(g, p, stream);
    }
    return CODEGEMM_UNSUPPORTED;
}

int launch_gemm_centroid_m1(const Geometry& g, const GemmParams& p, hipStream_t stream);
int launch_gemm_centroid_m2(const Geometry& g, const GemmParams& p, hipStream_t stream);
int launch_gemm_centroid_m3(const Geometry& g, const GemmParams& p, hipStream_t stream);
int launch_gemm_centroid_m4(const Geometry& g, const GemmParams& p, hipStream_t stream);

}  // namespace cg
