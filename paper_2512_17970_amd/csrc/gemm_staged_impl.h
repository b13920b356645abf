// The centroid kernel with codes and activations staged in LDS: fp16 output, one or two codebooks of short
// vectors; blocks of 128 rows, and from 5 batch rows on of 64 and 32.  Included by gemm_prompt_impl.h; table, lookups and columns as in gemm_centroid_impl.h.
//
// Why a second kernel.  The chip runs out of power before it runs out of anything else here: with lookups, MFMAs and the stream of
// codes at work its clock falls from 2.4 to 1.2-1.6 GHz (s_memtime against the 100 MHz counter; 8192->57344 v8 m2 with four rows
// takes 42 us on random and 25 us on all-zero operands), and a vector instruction beside a lookup and its MFMA costs its whole
// issue time (10 ns per lookup and SIMD + 1.75 ns per vector instruction).  So what counts is work per lookup.  A wavefront that
// loads its operands into registers pays for the layout there: either the columns are octets x sub-vectors (SB = 4, 2) and the
// result tile holds 4 or 2 times the elements that mean something, each to be picked and scaled for every group, or pairs of lanes
// exchange what they loaded (SB = 1).  Here the memory pipeline writes codes, x and scales to LDS by itself (buffer_load .. lds),
// in runs of 128 bytes that the lanes read back in any arrangement: all 16 columns are octets, an accumulator holds the whole
// contraction of its 16 x 16 tile, and neither loads nor exchanges take registers.  Vector instructions per lookup, v8 m2 g128,
// four rows: 4.1 -> 1.9.  The table lies at the start of the LDS and the rings behind it, so that an address is one byte-permute (the other
// way round cost an addition per lookup, 3 to 9 % of a call).
//
// Measured (us, back to back; before -> here): see staged_batch in plan.hip.
//
// Lower blocks (SPLIT = 2, 4).  The 16 columns are 8 octets x 2 halves or 4 octets x 4 quarters of their rows: lane (octet, part) reads the
// 4 or 2 bytes of its rows from the staged entry and takes 4 or 2 lookups per chunk, each of which feeds one MFMA for 16 batch rows whatever the
// height, where columns of octets x sub-vectors take two (64 rows) or four (32 rows) and discard as much of the result.  us, centroid
// kernel -> here: v8 m2 16 rows 4096^2 8.7 -> 5.8, 4096->6144 9.4 -> 5.9; 32 rows 14336->4096 18.8 -> 13.4; v4 m1 g128 8 rows 14336->4096 9.9 -> 7.9.
// Short groups (GS = 2): a round's 4 chunks are neighbours, so each round closes its sums with a scale of its own, a row's beside the MFMAs of
// the row after it; a stage's scales, one set per round, are one more request.  64-row blocks, v8 m1 g32 16 rows: 2.3 times the centroid kernel's speed.
// 16 wavefronts, of twice the K slices or of two row groups, are slower (5.9 -> 6.6, 6.2 us: each has the same code in front of and behind its
// loop), and so are three or four stages (5.7 -> 6.1 us, 8 rows) and stages of twice the size for two tiles of short codes (4 to 10 %).
//
// A wavefront's stage is 8 or 16 pieces of 16 bytes of the codes of each octet (two rounds of 4 chunks, four for v8 m1 and 32-row blocks), the
// x of these chunks and, with group scales, 16 bytes of scales per octet; it keeps D of them.  DMA instruction e of a stage takes 64 pieces: lane ->
// octet and place in its run, which holds piece place ^ turn(octet), so that the 16 lanes of a read, which take the same piece of all octets,
// touch different columns of 16 bytes (128 rows in the plain order, one octet per run of 64 bytes, is a 2-way conflict, and 64-byte runs stream
// 117 MB in 31 us where 128-byte runs take 24).  The lookups have no conflicts; those
// that are left, a tenth of the LDS cycles (v8 m2 g128, four rows, 128-row blocks), are in the reads of codes, two halves of 8 bytes, and of x.
// Only the wavefront itself reads its stages, so nothing but its own count of outstanding requests orders them: no barrier
// in the loop.  The compiler does not see these requests (inline assembly without outputs), and waits are written out.
//
// What a short call spends outside the loop is counted in requests and instructions: the memory pipeline takes 64 bytes of requests per clock,
// and code runs from a cold instruction cache.  So the codebooks come as they are, 2 to 8 KB, and the threads write the table's copies while
// stage 0 is on its way (the table by requests, 64 KB of them: 0.4 us); the other stages are asked for behind that; nothing is asked for past
// a slice's end; and a request is an addition and the instruction, without a branch of its own.  us, before -> with all of it: 4096->28672 v8 m2
// 16 rows 15.2 -> 13.3, v4 m1 g128 8 rows 11.0 -> 10.1; 8192->57344 v8 m2 g128 4 rows 40.2 -> 37.9.
#pragma once

#include "gemm_centroid_impl.h"

namespace cg {

typedef __attribute__((address_space(3))) u32x2_t lds_u2;
typedef __attribute__((address_space(3))) u32x4_t lds_u4;

// Descriptor of `bytes` bytes at `base` (uniform) as the four words that inline assembly takes.  The compiler does not count wait states
// into inline assembly, and a buffer instruction needs five behind a vector instruction that wrote its scalar operands.
__device__ __forceinline__ u32x4_t buffer_words(const void* base, int bytes)
{
    const uint64_t a = reinterpret_cast<uint64_t>(base);
    u32x4_t words = {(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a), (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xffffu)),
                     (uint32_t)__builtin_amdgcn_readfirstlane(bytes), 0x00020000u};
    asm volatile("s_nop 4" : "+s"(words));
    return words;
}

// 16 bytes per active lane from voff + soff of the buffer to LDS byte address lds + 16 lane.  A voff past the end of the
// buffer reads nothing, but counts as a request.  The LDS address goes through m0, which the compiler sets (as a clobber it would be
// kept just as safe, with a warning per request: the register is reserved); one wait state lies between.
template <bool STREAM>
__device__ __forceinline__ void load_to_lds(uint32_t lds, int voff, u32x4_t rsrc, int soff)
{
    if constexpr (STREAM) asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds" :: "{m0}"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
    else asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" :: "{m0}"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}

template <int N>
__device__ __forceinline__ void wait_requests() { asm volatile("s_waitcnt vmcnt(%0)" :: "i"(N) : "memory"); }

// Sizes of a wavefront's ring.  SPLIT: row groups of an octet (1, 2 or 4; blocks of 128, 64 or 32 rows); BR: batch rows of a tile (4, 8 or 16);
// NT: tiles (2: BR = 16); D: stages.
template <int M, int V, int GS, int SPLIT, int BR, int NT, int D>
struct StagedShape {
    static constexpr int kWaves = 8;
    static constexpr int kOctets = 16 / SPLIT;         // octets of a block
    static constexpr int kRows = 8 / SPLIT;            // rows of an octet that one lane takes
    static constexpr bool kHalf = V == 8 && M == 1;    // a piece holds two chunks
    static constexpr int kRounds = NT == 1 && (kHalf || SPLIT == 4) ? 4 : 2;   // rounds (4 chunks of 16 bytes of x) per stage
    static constexpr int kChunks = 4 * kRounds;
    static constexpr int kPieces = kHalf ? kChunks / 2 : kChunks;              // of an octet
    static constexpr int kCodeLoads = (kOctets * kPieces + 63) / 64;
    static constexpr int kXRows = 64 / kChunks;        // batch rows of a DMA instruction
    static constexpr int kXLoads = (NT * BR + kXRows - 1) / kXRows;
    static constexpr int kXAt = kOctets * kPieces * 16;                        // behind the codes
    static constexpr int kXTile = BR * kChunks * 16;
    static constexpr int kScalesAt = kXAt + NT * kXTile;
    static constexpr bool kZeros = BR == 8;            // a row of zeros for the batch rows that an MFMA has and the tile has not (4: copies do as well)
    static constexpr int kScales = GS == 2 ? kRounds : 1;                      // of a row: per round, or per step in its first stage
    static constexpr int kZeroAt = kScalesAt + (GS ? kScales * kOctets * 16 : 0);
    static constexpr int kStage = kZeroAt + (kZeros ? 16 : 0);
    static constexpr int kRing = kStage * D;
    // The rings lie behind the table: a lookup's address is then the byte-permute alone, without an addition per lookup.
    static constexpr int kRingAt = CentroidTable<M, V>::kBytes;
    // The codebooks as they come, from which the table is filled: behind the rings if there is room, else where the table will be.
    static constexpr int kRawBytes = M * kCentroids * V * 2;
    static constexpr bool kRawApart = kRingAt + kRing * kWaves + kRawBytes <= kMaxLds;
    static constexpr int kRawAt = kRawApart ? kRingAt + kRing * kWaves : 0;
    static constexpr int kLds = kRingAt + kRing * kWaves + (kRawApart ? kRawBytes : 0);
    static constexpr int kStep = 4 / kRounds;          // stages per step of 16 chunks
    // Piece `pos` of octet o lies at place pos ^ turn(o) of the octet's run, so that 16 lanes which take the same piece of all octets
    // touch different columns of 16 bytes (pieces of two octets share 256 bytes where a run is 128).
    static __host__ __device__ constexpr int turn(int o) { return (kPieces == 16 ? o : kPieces == 8 ? o >> 1 : o >> 2) * SPLIT & (kPieces - 1); }
    // Requests of stage t (counted from a step's first; scales come with that one), and of stages t .. t + n - 1.
    static constexpr int loads(int t) { return kCodeLoads + kXLoads + (GS == 2 || (GS == 1 && t % kStep == 0) ? 1 : 0); }
    static constexpr int loads(int t, int n) { int k = 0; for (int j = 0; j < n; ++j) k += loads(t + j); return k; }
    static constexpr int kTurn = D % 2 ? 2 * D : D;    // stages per turn of the loop: whole steps, registers in pairs
    // Waits until stage t + 1 has landed, stages t + 2 .. t + D being outstanding.
    template <int I = 0>
    static __device__ __forceinline__ void wait(int t)
    {
        if constexpr (I < kTurn) {
            if (t == I) wait_requests<loads(I + 2, D - 1)>();
            else wait<I + 1>(t);
        }
    }
    // Waits until all but the requests of stages FIRST .. FIRST + n - 1 (n at most D) have landed.
    template <int FIRST, int I = 0>
    static __device__ __forceinline__ void wait_but(int n)
    {
        if (I == D || n <= I) wait_requests<loads(FIRST, I)>();
        else if constexpr (I < D) wait_but<FIRST, I + 1>(n);
    }
};

template <int M, int V, int GS, int SPLIT, int BR, int NT, int D>
__global__ void __launch_bounds__(512) gemm_staged_kernel(CG_HEAD_PARAMS, const GemmParams pk)
{
    GemmParams p = with_head(pk, hx, hpacked, hcodebooks, hgscales, hK, hNKT, hKPW, hB, hNGR, hmisc);
    p.mem[0].N = hNGR;                                 // see the launch: N in place of the granules, and either kind of scales
    if constexpr (!GS) p.mem[0].scales = reinterpret_cast<const _Float16*>(hgscales);
    typedef CentroidTable<M, V> T;
    typedef StagedShape<M, V, GS, SPLIT, BR, NT, D> S;
    static_assert((V == 8 && M <= 2) || (V == 4 && M == 1), "the table takes 64 KB, a chunk 8 or 16 bytes of codes");
    static_assert(GS <= 2, "0 one scale per row, 1 a step of 16 chunks lies in one group, 2 groups of 4 or 8 chunks");
    static_assert(NT == 1 || BR == 16, "tiles of 16 rows");
    constexpr int KW = S::kWaves, THREADS = KW * kWave, OCT = S::kOctets, U = S::kRows, RB = 8 * OCT;
    constexpr int BT = BR * NT;
    constexpr int R = S::kRounds;
    constexpr int SPU = (V == 4 ? 4 : 8) / R;          // stages per unit of 32 sub-vectors
    constexpr int SPS = S::kStep;                      // .. per step of 16 chunks
    constexpr int NSB = R * M;                         // (round, codebook) of a stage: U lookups and U NT MFMAs each
    constexpr int WR = (V == 4 ? 2 : M) * (SPLIT == 1 ? 2 : 1);            // registers of codes per lane and round
    constexpr int kUnitBytes = kGranuleRows * kSlots * M;
    constexpr int kOutOfRange = 0x7ffffff0;

    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ks = blockIdx.x;
    const Member mm = member_of(p, blockIdx.y);
    const int blk = blockIdx.y - mm.blk0;
    const int gr = blk * RB / kGranuleRows, oct0 = blk % SPLIT * OCT;      // granule, and the block's first octet in it
    const int b0 = blockIdx.z * BT;
    const int kt0 = ks * p.KPW;
    const int nq = min(p.KPW, p.NKT - kt0);
    const int q = lane >> 4, i16 = lane & 15;
    const int oct = i16 & (OCT - 1), rg = i16 / OCT;   // the lane's column: rows U rg .. of octet oct
    const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>((lds_float*)smem);
    const uint32_t ring = lds0 + (uint32_t)(S::kRingAt + wave * S::kRing);

    // This wavefront's stages of the workgroup's K range (whole steps with group scales).
    constexpr int ALIGN = GS == 1 ? SPS : 1;
    const int total = nq * SPU / ALIGN;
    const int s_beg = total * wave / KW * ALIGN, s_end = total * (wave + 1) / KW * ALIGN;

    // Row scales, in front of all requests that are counted; then the codebooks, for which everything waits.
    uint32_t scale_bits = 0x3c00u;
    if constexpr (!GS) scale_bits = row_scale_bits<RB>(mm, tid, blk);
    if (wave < S::kRawBytes / 1024)
        load_to_lds<false>(lds0 + (uint32_t)(S::kRawAt + wave * 1024), wave * 1024 + lane * 16, buffer_words(mm.codebooks, S::kRawBytes), 0);

    constexpr int kOctetBytes = kSlots * 8 * M;
    const u32x4_t c_rsrc = buffer_words(mm.packed + ((size_t)gr * p.NKT + kt0) * kUnitBytes + oct0 * kOctetBytes, nq * kUnitBytes - oct0 * kOctetBytes);
    const u32x4_t x_rsrc = buffer_words(p.x + (size_t)b0 * p.K, min(p.B - b0, BT) * p.K * 2);
    u32x4_t s_rsrc = {};
    if constexpr (GS) s_rsrc = buffer_words(mm.gscales + ((size_t)gr * p.NKT + kt0) * p.GPU * 256 + oct0 * 16, nq * p.GPU * 256 - oct0 * 16);
    const int x_el0 = kt0 * kSlots * V;
    int c_voff[S::kCodeLoads], x_voff[S::kXLoads];
#pragma unroll
    for (int e = 0; e < S::kCodeLoads; ++e) {
        const int o = (64 * e + lane) / S::kPieces, piece = (lane & (S::kPieces - 1)) ^ S::turn(o);
        c_voff[e] = o * kOctetBytes + piece * 16;
    }
#pragma unroll
    for (int e = 0; e < S::kXLoads; ++e) {
        const int row = e * S::kXRows + lane / S::kChunks;
        x_voff[e] = row * p.K * 2 + ((lane & (S::kChunks - 1)) ^ ((row & 15) / (16 / S::kChunks))) * 16;
    }
    constexpr int SUBS = V == 4 ? 2 : 1;               // sub-vectors of a chunk
    const int s_voff = GS == 2 ? ((lane / OCT * (4 * SUBS)) >> p.gshift) * 256 + lane % OCT * 16 : 0;     // scales of round lane / OCT
    // Stage s into its slot.
    auto request = [&](int s, int t) {                 // t = s - s_beg, or as much as matters of it
        const uint32_t at = ring + (uint32_t)(t % D * S::kStage);
        const int x0 = x_el0 + s * (S::kChunks * 8);
        const int off = (s / SPU) * kUnitBytes + (s % SPU) * (S::kPieces * 16);
#pragma unroll
        for (int e = 0; e < S::kCodeLoads; ++e) {
            constexpr int LANES = OCT * S::kPieces;
            if (LANES >= 64 || lane < LANES) load_to_lds<true>(at + e * 1024, c_voff[e], c_rsrc, off);
        }
        const int x_add = x0 < p.K ? x0 * 2 : kOutOfRange & ~0xfffffff;     // a row's end reaches into the next row, the last one's past the buffer
#pragma unroll
        for (int e = 0; e < S::kXLoads; ++e) {
            constexpr int LANES = BT < S::kXRows ? BT * S::kChunks : 64;
            if (LANES == 64 || lane < LANES) load_to_lds<false>(at + S::kXAt + e * 1024, x_voff[e] + x_add, x_rsrc, 0);
        }
        if constexpr (GS == 2) {                       // a group of 4 or 8 chunks: a stage begins with one
            const int unit_group = ((s % SPU) * (S::kChunks * SUBS)) >> p.gshift;
            if (lane < S::kScales * OCT) load_to_lds<false>(at + S::kScalesAt, s_voff, s_rsrc, ((s / SPU) * p.GPU + unit_group) * 256);
        } else if (GS && t % SPS == 0) {
            const int sub = V == 4 ? 0 : (s % SPU) / SPS * 16;             // first sub-vector of the step in its unit
            if (lane < OCT) load_to_lds<false>(at + S::kScalesAt, lane * 16, s_rsrc, ((s / SPU) * p.GPU + (sub >> p.gshift)) * 256);
        }
    };
    if constexpr (S::kZeros) {
        if (lane < 4 * D) *reinterpret_cast<lds_u32*>(static_cast<uintptr_t>(ring + (uint32_t)(lane / 4 * S::kStage + S::kZeroAt + lane % 4 * 4))) = 0;
    }
    const int stages = s_end - s_beg, asked = min(stages, D);
    if (asked > 0) request(s_beg, 0);

    // The table: a centroid repeated in its columns, which start at another one in every row so that a wavefront's stores spread over the banks.
    S::template wait_but<0>(min(asked, 1));
    __syncthreads();
    {
        constexpr int TPE = THREADS / (M * kCentroids);                    // threads that share one centroid's columns
        typedef typename Frag<V == 4 ? 4 : 16>::type entry_t;              // 8 or 16 bytes
        typedef __attribute__((address_space(3))) entry_t lds_entry;
        const int c = tid / TPE / kCentroids, code = tid / TPE % kCentroids;
        constexpr int COLS = T::columns(0), MINE = COLS / TPE;
        const entry_t fill = *reinterpret_cast<const lds_entry*>(static_cast<uintptr_t>(lds0 + (uint32_t)(S::kRawAt + tid / TPE * V * 2)));
        if constexpr (!S::kRawApart) __syncthreads();  // everyone has its centroid: the table takes their place
        const uint32_t first = lds0 + (uint32_t)(code * 256 + c * 128 + (tid % TPE * MINE + (tid / TPE & (MINE - 1))) * T::kEntry);
#pragma unroll
        for (int j = 0; j < MINE; ++j) *reinterpret_cast<lds_entry*>(static_cast<uintptr_t>(first ^ (uint32_t)(j * T::kEntry))) = fill;
    }
#pragma unroll
    for (int d = 1; d < D; ++d)
        if (d < asked) request(s_beg + d, d);

    float4_t acc[NT][U];
    float4_t sum[GS ? NT : 1][GS ? U : 1];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            acc[nt][u] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
            if constexpr (GS) sum[nt][u] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
        }

    // Lookup bases: two codebooks share a row of the table, and lanes 8..15 of 16 take them in the opposite order.
    const int order = M == 2 ? (lane >> 3) & 1 : 0;
    uint32_t base[M];
#pragma unroll
    for (int k = 0; k < M; ++k) base[k] = lds0 + (uint32_t)((M == 2 ? (k ^ order) * 128 : 0) + (lane & (T::columns(k) - 1)) * T::kEntry);
    // Where the lane finds the codes of its rows, chunk 4 r + q, and x of batch row i16 % BR, the same chunk.
    uint32_t c_at[R], c_at2[R], x_at[R];
    const int xr = i16 & (BR - 1);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int chunk = 4 * r + q, piece = S::kHalf ? chunk >> 1 : chunk;
        c_at[r] = ring + (uint32_t)((oct * S::kPieces + (piece ^ S::turn(oct))) * 16 + (S::kHalf ? (chunk & 1) * 8 : order * 8) + rg * U);
        c_at2[r] = c_at[r] ^ 8u;                       // the other codebook's
        x_at[r] = ring + (uint32_t)(S::kZeros && i16 >= BR ? S::kZeroAt : (xr * S::kChunks + (chunk ^ (xr / (16 / S::kChunks)))) * 16 + S::kXAt);
    }
    const uint32_t s_at = ring + (uint32_t)(S::kScalesAt + oct * 16 + rg * (U * 2));
    // Codes of U rows: 8, 4 or 2 bytes.
    auto read_rows = [&](uint32_t* w, uint32_t at) {
        if constexpr (SPLIT == 1) {
            const u32x2_t a = *reinterpret_cast<const lds_u2*>(static_cast<uintptr_t>(at));
            w[0] = a.x; w[1] = a.y;
        } else if constexpr (SPLIT == 2) w[0] = *reinterpret_cast<const lds_u32*>(static_cast<uintptr_t>(at));
        else w[0] = *reinterpret_cast<const lds_u16*>(static_cast<uintptr_t>(at));
    };
    auto read_codes = [&](uint32_t (&w)[R][WR], int d) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t at = c_at[r] + (uint32_t)(d * S::kStage);
            if constexpr (V == 4 && SPLIT == 1) {
                const u32x4_t a = *reinterpret_cast<const lds_u4*>(static_cast<uintptr_t>(at));
                w[r][0] = a.x; w[r][1] = a.y; w[r][2] = a.z; w[r][3] = a.w;
            } else {
                read_rows(w[r], at);
                if constexpr (V == 4) read_rows(w[r] + WR / 2, at + 8);
                else if constexpr (M == 2) read_rows(w[r] + WR / 2, c_at2[r] + (uint32_t)(d * S::kStage));
            }
        }
    };
    typedef _Float16 scales_t __attribute__((ext_vector_type(S::kRows)));
    typedef __attribute__((address_space(3))) scales_t lds_scales;
    auto read_x = [&](half8_t (&x)[R][NT], int d, int s) {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                x[r][nt] = *reinterpret_cast<const lds_half8*>(static_cast<uintptr_t>(x_at[r] + (uint32_t)(d * S::kStage + nt * S::kXTile)));
        if (x_el0 + (s + 1) * (S::kChunks * 8) > p.K) {    // the stage reaches past the end of the rows
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int left = p.K - (x_el0 + s * (S::kChunks * 8) + (4 * r + q) * 8);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    u32x4_t t = __builtin_bit_cast(u32x4_t, x[r][nt]);
                    t.x = left > 0 ? t.x : 0u; t.y = left > 0 ? t.y : 0u; t.z = left > 4 ? t.z : 0u; t.w = left > 4 ? t.w : 0u;
                    x[r][nt] = __builtin_bit_cast(half8_t, t);
                }
            }
        }
    };
    // Centroid operand of MFMA u in (round, codebook) k of a stage: row U rg + u of the lane's octet.
    auto fetch = [&](const uint32_t (&w)[R][WR], int k, int u) -> half8_t {
        const int c = k % M, r = k / M;
        const uint32_t sel = 0x0c020000u | (uint32_t)(4 + u % 4) << 8;
        if constexpr (V == 4) {
            const half4_t lo4 = *reinterpret_cast<const lds_half4*>(static_cast<uintptr_t>(__builtin_amdgcn_perm(w[r][u / 4], base[0], sel)));
            const half4_t hi4 = *reinterpret_cast<const lds_half4*>(static_cast<uintptr_t>(__builtin_amdgcn_perm(w[r][WR / 2 + u / 4], base[0], sel)));
            return __builtin_shufflevector(lo4, hi4, 0, 1, 2, 3, 4, 5, 6, 7);
        } else {
            return *reinterpret_cast<const lds_half8*>(static_cast<uintptr_t>(__builtin_amdgcn_perm(w[r][c * (WR / M) + u / 4], base[c], sel)));
        }
    };
    auto add_scaled = [&](const scales_t& scales, int u) {
        const float f = (float)scales[u];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[GS ? nt : 0][GS ? u : 0][e] = __builtin_fmaf(f, acc[nt][u][e], sum[GS ? nt : 0][GS ? u : 0][e]);
    };
    auto read_scales = [&](scales_t (&dst)[S::kScales], int d) {
#pragma unroll
        for (int r = 0; r < S::kScales; ++r) dst[r] = *reinterpret_cast<const lds_scales*>(static_cast<uintptr_t>(s_at + (uint32_t)(d * S::kStage + r * OCT * 16)));
    };

    S::template wait_but<1>(asked - 1);                // the first stage
    __syncthreads();                                   // the table

    // Main loop.  While stage s is multiplied, codes and x of stage s + 1 come from LDS to registers, and its slot is asked
    // for again as soon as they have.  Every MFMA is followed by the lookup that takes its operand's registers, AHEAD lookups later.
    constexpr int LOOKUPS = NSB * U, AHEAD = LOOKUPS < 8 ? LOOKUPS : 8;
    uint32_t w[2][R][WR];
    half8_t xv[2][R][NT], a[AHEAD];
    scales_t scales[S::kScales], scales_next[S::kScales];
    read_codes(w[0], 0);
    read_x(xv[0], 0, s_beg);
    if constexpr (GS) read_scales(scales_next, 0);
#pragma unroll
    for (int n = 0; n < AHEAD; ++n) a[n] = fetch(w[0], n / U, n % U);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // slot 0 has been read
    if (D < stages) request(s_beg + D, D);
    constexpr int TURN = S::kTurn;
    for (int s0 = s_beg; s0 < s_end; s0 += TURN) {
#pragma unroll
        for (int t = 0; t < TURN; ++t) {
            const int s = s0 + t, n = (t + 1) % D;
            if (s < s_end) {
                const bool opens = GS == 2 || (GS && t % SPS == 0), closes = GS == 2 || (GS && t % SPS == SPS - 1);   // of a step
                if (opens) {
#pragma unroll
                    for (int r = 0; r < S::kScales; ++r) scales[r] = scales_next[r];
                }
                if (s + D < s_end) S::wait(t);         // stage s + 1 has landed
                else wait_requests<0>();
                read_codes(w[(t + 1) & 1], n);
                read_x(xv[(t + 1) & 1], n, s + 1);
                if (closes) read_scales(scales_next, n);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int l = 0; l < LOOKUPS; ++l) {
                    const int k = l / U, u = l % U, next = l + AHEAD;
                    const bool first = GS == 2 ? k % M == 0 : opens && k == 0;
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        acc[nt][u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xv[t & 1][k / M][nt], a[l % AHEAD], first ? float4_t{} : acc[nt][u], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);             // the lookup after its operand's last use: no second set of registers
                    a[l % AHEAD] = next < LOOKUPS ? fetch(w[t & 1], next / U, next % U) : fetch(w[(t + 1) & 1], (next - LOOKUPS) / U, next % U);
                    if constexpr (GS == 2) {           // a row's sum is scaled beside the MFMAs of the row after it
                        if (u > 0 && k % M == M - 1) add_scaled(scales[k / M], u - 1);
                        if (u == 0 && k % M == 0 && k > 0) add_scaled(scales[k / M - 1], U - 1);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                // the values are here: what they were read from may be overwritten
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) asm volatile("" : "+v"(xv[(t + 1) & 1][r][nt]));
                if (closes) {
#pragma unroll
                    for (int r = 0; r < S::kScales; ++r) asm volatile("" : "+v"(scales_next[r]));
                }
                if (s + 1 + D < s_end) request(s + 1 + D, t + 1 + D);
                if (closes) {
#pragma unroll
                    for (int u = GS == 2 ? U - 1 : 0; u < U; ++u) add_scaled(scales[S::kScales - 1], u);
                }
            }
        }
    }

    // Sum over the wavefronts' K slices as in the centroid kernel.  Lane (i16, q): its U rows, batch rows 16 nt + 4 q + e.
    typedef SliceSums<THREADS, BT, RB, KW> Sums;
    float* parts = reinterpret_cast<float*>(smem);
    __syncthreads();                                    // everyone is done with the table
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int b = 4 * q + e;
            if (b < BR && b0 + BR * nt + b < p.B) {
                float* dst = parts + (wave * BT + BR * nt + b) * Sums::kStride + oct * 8 + rg * U;
                typedef float rows_t __attribute__((ext_vector_type(U > 4 ? 4 : U)));
                constexpr int W = U > 4 ? 4 : U;
#pragma unroll
                for (int u = 0; u < U; u += W) {
                    rows_t v;
#pragma unroll
                    for (int k = 0; k < W; ++k) v[k] = GS ? sum[GS ? nt : 0][GS ? u + k : 0][e] : acc[nt][u + k][e];
                    *reinterpret_cast<rows_t*>(dst + u) = v;
                }
            }
        }
    Sums::finish(p, mm, parts, scale_bits, tid, blk, ks, b0);
}

template <int M, int V, int GS, int SPLIT, int BR, int NT, int D>
int launch_gemm_staged_one(const Geometry& g, const GemmParams& p, hipStream_t stream)
{
    auto fn = gemm_staged_kernel<M, V, GS, SPLIT, BR, NT, D>;
    typedef StagedShape<M, V, GS, SPLIT, BR, NT, D> S;
    constexpr int RB = kGranuleRows / SPLIT;
    if (g.RB != RB || g.BG != BR * NT) return CODEGEMM_UNSUPPORTED;
    constexpr size_t stage = SliceSums<S::kWaves * kWave, BR * NT, RB, S::kWaves>::kLds;
    constexpr size_t lds = stage > S::kLds ? stage : S::kLds;
    static_assert(lds <= (size_t)kMaxLds, "LDS");
    int st = set_max_lds(reinterpret_cast<const void*>(fn), lds);
    if (st != CODEGEMM_OK) return st;
    const dim3 grid((unsigned)g.NKS, (unsigned)g.NBLK, (unsigned)g.NG);
    const uint8_t* scales = GS ? p.mem[0].gscales : reinterpret_cast<const uint8_t*>(p.mem[0].scales);
    hipLaunchKernelGGL(fn, grid, dim3(S::kWaves * kWave), lds, stream, CG_HEAD_ARGS_WITH(p, scales, p.mem[0].N), p);
    return hipGetLastError() == hipSuccess ? CODEGEMM_OK : CODEGEMM_LAUNCH_FAILED;
}

// Two stages everywhere: three or four are no faster (v8 m2 g128, four rows, 8192->28672: 19.1, 19.5 us with four) and leave less
// room for batch rows.
template <int M, int V, int GS>
int launch_gemm_staged(const Geometry& g, const GemmParams& p, hipStream_t stream)
{
    constexpr bool WIDE = V == 8 && M == 1;
    if (g.RB == 64) {
        switch (g.BG) {
            case 8: return launch_gemm_staged_one<M, V, GS, 2, 8, 1, 2>(g, p, stream);
            case 16: return launch_gemm_staged_one<M, V, GS, 2, 16, 1, 2>(g, p, stream);
            case 32: if constexpr (!WIDE) return launch_gemm_staged_one<M, V, GS, 2, 16, 2, 2>(g, p, stream);
        }
        return CODEGEMM_UNSUPPORTED;
    }
    if (g.RB == 32) {
        switch (g.BG) {
            case 8: return launch_gemm_staged_one<M, V, GS, 4, 8, 1, 2>(g, p, stream);
            case 16: return launch_gemm_staged_one<M, V, GS, 4, 16, 1, 2>(g, p, stream);
            case 32: if constexpr (!WIDE) return launch_gemm_staged_one<M, V, GS, 4, 16, 2, 2>(g, p, stream);
        }
        return CODEGEMM_UNSUPPORTED;
    }
    switch (g.BG) {
        case 4:
            if constexpr (GS == 1) return launch_gemm_staged_one<M, V, GS, 1, 4, 1, 2>(g, p, stream);
            break;
        case 8:
            if constexpr (GS == 1 && WIDE) return launch_gemm_staged_one<M, V, GS, 1, 8, 1, 2>(g, p, stream);
            break;
        case 16:
            if constexpr (GS == 0 || !WIDE) return launch_gemm_staged_one<M, V, GS, 1, 16, 1, 2>(g, p, stream);
            break;
        case 32:
            if constexpr (GS == 0 && !WIDE) return launch_gemm_staged_one<M, V, GS, 1, 16, 2, 2>(g, p, stream);
            break;
    }
    return CODEGEMM_UNSUPPORTED;
}

}  // namespace cg
