// The centroid kernel with codes and activations staged in LDS: blocks of 128 rows, fp16 output, one or two codebooks of short
// vectors.  Included by gemm_prompt_impl.h; table, lookups and columns as in gemm_centroid_impl.h.
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
// A wavefront's stage is 8 pieces of 16 bytes of the codes of each of the 16 octets (two rounds of 4 chunks, four for v8 m1), the
// x of these chunks and, with group scales, 256 bytes of scales; it keeps D of them.  DMA instruction e of a stage takes octets
// 8 e .. 8 e + 7: lane -> octet 8 e + lane / 8, piece (lane % 8) ^ (octet / 2), which lands at place `lane`, so that the 16 lanes
// of a read, which take the same piece of 16 octets, touch 16 different columns of 16 bytes (one octet per run of 64 bytes, the
// plain order, is a 2-way conflict, and 64-byte runs stream 117 MB in 31 us where 128-byte runs take 24).  The lookups have no conflicts; those
// that are left, a tenth of the LDS cycles (v8 m2 g128, four rows), are in the reads of codes, two halves of 8 bytes, and of x.
// Only the wavefront itself reads its stages, so nothing but its own count of outstanding requests orders them: no barrier
// in the loop.  The compiler does not see these requests (inline assembly without outputs), and waits are written out.
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

// Sizes of a wavefront's ring.  BR: batch rows of a tile (4, 8 or 16); NT: tiles (2: BR = 16); D: stages.
template <int M, int V, int GS, int BR, int NT, int D>
struct StagedShape {
    static constexpr int kWaves = 8;
    static constexpr bool kHalf = V == 8 && M == 1;    // a piece holds two chunks
    static constexpr int kRounds = kHalf ? 4 : 2;      // rounds (4 chunks of 16 bytes of x) per stage
    static constexpr int kChunks = 4 * kRounds;
    static constexpr int kXRows = 64 / kChunks;        // batch rows of a DMA instruction
    static constexpr int kXLoads = (NT * BR + kXRows - 1) / kXRows;
    static constexpr int kXAt = 2048;                  // behind the codes
    static constexpr int kXTile = BR * kChunks * 16;
    static constexpr int kScalesAt = kXAt + NT * kXTile;
    static constexpr int kStage = kScalesAt + (GS ? 256 : 0);
    static constexpr int kRing = kStage * D;
    // The rings lie behind the table: a lookup's address is then the byte-permute alone, without an addition per lookup.
    static constexpr int kRingAt = CentroidTable<M, V>::kBytes;
    static constexpr int kLds = kRingAt + kRing * kWaves;
    static constexpr int kStep = 4 / kRounds;          // stages per step of 16 chunks
    // Requests of stage t (counted from a step's first; scales come with that one), and of stages t .. t + n - 1.
    static constexpr int loads(int t) { return 2 + kXLoads + (GS && t % kStep == 0 ? 1 : 0); }
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
};

template <int M, int V, int GS, int BR, int NT, int D>
__global__ void __launch_bounds__(512) gemm_staged_kernel(CG_HEAD_PARAMS, const GemmParams pk)
{
    const GemmParams p = with_head(pk, hx, hpacked, hcodebooks, hgscales, hK, hNKT, hKPW, hB, hNGR, hmisc);
    typedef CentroidTable<M, V> T;
    typedef StagedShape<M, V, GS, BR, NT, D> S;
    static_assert((V == 8 && M <= 2) || (V == 4 && M == 1), "the table takes 64 KB, a chunk 8 or 16 bytes of codes");
    static_assert(GS <= 1, "a step of 16 chunks lies in one group");
    static_assert(NT == 1 || BR == 16, "tiles of 16 rows");
    constexpr int KW = S::kWaves, THREADS = KW * kWave, RB = kGranuleRows;
    constexpr int BT = BR * NT;
    constexpr int R = S::kRounds;
    constexpr int SPU = (V == 4 ? 4 : 8) / R;          // stages per unit of 32 sub-vectors
    constexpr int SPS = S::kStep;                      // .. per step of 16 chunks
    constexpr int NSB = R * M;                         // (round, codebook) of a stage: 8 lookups and 8 NT MFMAs each
    constexpr int WR = V == 4 ? 4 : 2 * M;             // dwords of codes per lane and round
    constexpr int kUnitBytes = kGranuleRows * kSlots * M;
    constexpr int kOutOfRange = 0x7ffffff0;

    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ks = blockIdx.x;
    const Member mm = member_of(p, blockIdx.y);
    const int blk = blockIdx.y - mm.blk0;              // = the granule
    const int b0 = blockIdx.z * BT;
    const int kt0 = ks * p.KPW;
    const int nq = min(p.KPW, p.NKT - kt0);
    const int q = lane >> 4, i16 = lane & 15;
    const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>((lds_float*)smem);
    const uint32_t ring = lds0 + (uint32_t)(S::kRingAt + wave * S::kRing);

    // This wavefront's stages of the workgroup's K range (whole steps with group scales).
    constexpr int ALIGN = GS ? SPS : 1;
    const int total = nq * SPU / ALIGN;
    const int s_beg = total * wave / KW * ALIGN, s_end = total * (wave + 1) / KW * ALIGN;

    // The table, requested first: everything waits for it.  A row is copied into its columns on the way (v = 4: centroids of 8
    // bytes, which a request cannot repeat, come as they are).
    if constexpr (V == 8) {
        const u32x4_t t_rsrc = buffer_words(mm.codebooks, M * kCentroids * V * 2);
#pragma unroll
        for (int k = 0; k < T::kBytes / 1024 / KW; ++k) {
            const int at = (k * KW + wave) * 1024;
            const int code = at / 256 + (lane >> 4), c = M == 2 ? (lane & 15) >> 3 : 0;
            load_to_lds<false>(lds0 + (uint32_t)at, (c * kCentroids + code) * 16, t_rsrc, 0);
        }
    } else if (wave < M * kCentroids * V * 2 / 1024) {
        load_to_lds<false>(lds0 + (uint32_t)(wave * 1024), wave * 1024 + lane * 16, buffer_words(mm.codebooks, M * kCentroids * V * 2), 0);
    }

    const u32x4_t c_rsrc = buffer_words(mm.packed + ((size_t)blk * p.NKT + kt0) * kUnitBytes, nq * kUnitBytes);
    const u32x4_t x_rsrc = buffer_words(p.x + (size_t)b0 * p.K, min(p.B - b0, BT) * p.K * 2);
    u32x4_t s_rsrc = {};
    if constexpr (GS) s_rsrc = buffer_words(mm.gscales + ((size_t)blk * p.NKT + kt0) * p.GPU * 256, nq * p.GPU * 256);
    const int x_el0 = kt0 * kSlots * V;
    int c_voff[2], x_voff[S::kXLoads];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int o = 8 * e + (lane >> 3), piece = (lane & 7) ^ (o >> 1);
        c_voff[e] = o * (kSlots * 8 * M) + piece * 16;
    }
#pragma unroll
    for (int e = 0; e < S::kXLoads; ++e) {
        const int row = e * S::kXRows + lane / S::kChunks;
        x_voff[e] = row * p.K * 2 + ((lane & (S::kChunks - 1)) ^ ((row & 15) / (16 / S::kChunks))) * 16;
    }
    // Stage s into its slot; past the end of the range the same number of requests, for nothing.
    auto request = [&](int s, int t) {                 // t = s - s_beg, or as much as matters of it
        const uint32_t at = ring + (uint32_t)(t % D * S::kStage);
        const int x0 = x_el0 + s * (S::kChunks * 8);
        const bool in = s < s_end;
        if (in) {
            const int off = (s / SPU) * kUnitBytes + (s % SPU) * 128;
#pragma unroll
            for (int e = 0; e < 2; ++e) load_to_lds<true>(at + e * 1024, c_voff[e], c_rsrc, off);
        } else {
#pragma unroll
            for (int e = 0; e < 2; ++e) load_to_lds<false>(at + e * 1024, kOutOfRange, c_rsrc, 0);
        }
        const bool some = in && x0 < p.K, whole = in && x0 + S::kChunks * 8 <= p.K;
#pragma unroll
        for (int e = 0; e < S::kXLoads; ++e) {
            constexpr int LANES = BT < S::kXRows ? BT * S::kChunks : 64;
            if (LANES == 64 || lane < LANES) {
                if (whole) load_to_lds<false>(at + S::kXAt + e * 1024, x_voff[e], x_rsrc, x0 * 2);
                else load_to_lds<false>(at + S::kXAt + e * 1024, some ? x_voff[e] + x0 * 2 : kOutOfRange, x_rsrc, 0);
            }
        }
        if (GS && t % SPS == 0) {
            const int sub = V == 4 ? 0 : (s % SPU) / SPS * 16;             // first sub-vector of the step in its unit
            if (lane < 16) {
                if (in) load_to_lds<false>(at + S::kScalesAt, lane * 16, s_rsrc, ((s / SPU) * p.GPU + (sub >> p.gshift)) * 256);
                else load_to_lds<false>(at + S::kScalesAt, kOutOfRange, s_rsrc, 0);
            }
        }
    };
#pragma unroll
    for (int d = 0; d < D; ++d) request(s_beg + d, d);
    uint32_t scale_bits = 0x3c00u;
    if constexpr (!GS) scale_bits = row_scale_bits<RB>(mm, tid, blk);

    if constexpr (V == 4) {
        wait_requests<S::loads(0, D)>();
        __syncthreads();
        // two threads per centroid, columns rotated by row so that a wavefront's stores spread over the banks
        const half4_t c = *reinterpret_cast<const lds_half4*>(static_cast<uintptr_t>(lds0 + (uint32_t)(tid / 2 * 8)));
        __syncthreads();                               // everyone has its centroid: the table takes their place
        const uint32_t row = lds0 + (uint32_t)(tid / 2 * 256);
#pragma unroll
        for (int j = 0; j < 16; ++j)
            *reinterpret_cast<lds_half4*>(static_cast<uintptr_t>(row + (uint32_t)(((tid & 1) * 16 + tid / 2 + j) & 31) * 8)) = c;
        static_assert(V != 4 || THREADS == 2 * kCentroids * M, "two threads per centroid");
    }

    float4_t acc[NT][8];
    float4_t sum[GS ? NT : 1][GS ? 8 : 1];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            acc[nt][u] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
            if constexpr (GS) sum[nt][u] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
        }

    // Lookup bases: two codebooks share a row of the table, and lanes 8..15 of 16 take them in the opposite order.
    const int order = M == 2 ? (lane >> 3) & 1 : 0;
    uint32_t base[M];
#pragma unroll
    for (int k = 0; k < M; ++k) base[k] = lds0 + (uint32_t)((M == 2 ? (k ^ order) * 128 : 0) + (lane & (T::columns(k) - 1)) * T::kEntry);
    // Where the lane finds the codes of octet i16, chunk 4 r + q, and x of batch row i16 % BR, the same chunk.
    uint32_t c_at[R], x_at[R];
    const int xr = i16 & (BR - 1);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int chunk = 4 * r + q, piece = S::kHalf ? chunk >> 1 : chunk;
        c_at[r] = ring + (uint32_t)(((i16 >> 3) * 64 + (i16 & 7) * 8 + (piece ^ (i16 >> 1))) * 16 + (S::kHalf ? (chunk & 1) * 8 : order * 8));
        x_at[r] = ring + (uint32_t)((xr * S::kChunks + (chunk ^ (xr / (16 / S::kChunks)))) * 16 + S::kXAt);
    }
    const uint32_t s_at = ring + (uint32_t)(S::kScalesAt + i16 * 16);
    auto read_codes = [&](uint32_t (&w)[R][WR], int d) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t at = c_at[r] + (uint32_t)(d * S::kStage);
            if constexpr (V == 4) {
                const u32x4_t a = *reinterpret_cast<const lds_u4*>(static_cast<uintptr_t>(at));
                w[r][0] = a.x; w[r][1] = a.y; w[r][2] = a.z; w[r][3] = a.w;
            } else {
                const u32x2_t a = *reinterpret_cast<const lds_u2*>(static_cast<uintptr_t>(at));
                w[r][0] = a.x; w[r][1] = a.y;
                if constexpr (M == 2) {
                    const u32x2_t b = *reinterpret_cast<const lds_u2*>(static_cast<uintptr_t>((c_at[r] ^ 8u) + (uint32_t)(d * S::kStage)));
                    w[r][2] = b.x; w[r][3] = b.y;
                }
            }
        }
    };
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
    // Centroid operand of MFMA u in (round, codebook) k of a stage: row u of the lane's octet.
    auto fetch = [&](const uint32_t (&w)[R][WR], int k, int u) -> half8_t {
        const int c = k % M, r = k / M;
        const uint32_t sel = 0x0c020000u | (uint32_t)(4 + u % 4) << 8;
        if constexpr (V == 4) {
            const half4_t lo4 = *reinterpret_cast<const lds_half4*>(static_cast<uintptr_t>(__builtin_amdgcn_perm(w[r][u / 4], base[0], sel)));
            const half4_t hi4 = *reinterpret_cast<const lds_half4*>(static_cast<uintptr_t>(__builtin_amdgcn_perm(w[r][2 + u / 4], base[0], sel)));
            return __builtin_shufflevector(lo4, hi4, 0, 1, 2, 3, 4, 5, 6, 7);
        } else {
            return *reinterpret_cast<const lds_half8*>(static_cast<uintptr_t>(__builtin_amdgcn_perm(w[r][2 * c + u / 4], base[c], sel)));
        }
    };
    auto add_scaled = [&](const half8_t& scales) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float f = (float)scales[u];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[GS ? nt : 0][GS ? u : 0][e] = __builtin_fmaf(f, acc[nt][u][e], sum[GS ? nt : 0][GS ? u : 0][e]);
        }
    };

    wait_requests<S::loads(1, D - 1)>();               // the table and the first stage
    __syncthreads();

    // Main loop.  While stage s is multiplied, codes and x of stage s + 1 come from LDS to registers, and its slot is asked
    // for again as soon as they have.  Every MFMA is followed by the lookup that takes its operand's registers, for the same
    // row of the next (round, codebook).
    uint32_t w[2][R][WR];
    half8_t xv[2][R][NT], scales, scales_next, a[8];
    read_codes(w[0], 0);
    read_x(xv[0], 0, s_beg);
    if constexpr (GS) scales_next = *reinterpret_cast<const lds_half8*>(static_cast<uintptr_t>(s_at));
#pragma unroll
    for (int u = 0; u < 8; ++u) a[u] = fetch(w[0], 0, u);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // slot 0 has been read
    request(s_beg + D, D);
    constexpr int U = S::kTurn;
    for (int s0 = s_beg; s0 < s_end; s0 += U) {
#pragma unroll
        for (int t = 0; t < U; ++t) {
            const int s = s0 + t, n = (t + 1) % D;
            if (s < s_end) {
                const bool opens = GS && t % SPS == 0, closes = GS && t % SPS == SPS - 1;   // of a step
                if (opens) scales = scales_next;
                S::wait(t);                            // stage s + 1 has landed
                read_codes(w[(t + 1) & 1], n);
                read_x(xv[(t + 1) & 1], n, s + 1);
                if (closes) scales_next = *reinterpret_cast<const lds_half8*>(static_cast<uintptr_t>(s_at + (uint32_t)(n * S::kStage)));
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int k = 0; k < NSB; ++k) {
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt)
                            acc[nt][u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xv[t & 1][k / M][nt], a[u], opens && k == 0 ? float4_t{} : acc[nt][u], 0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);             // the lookup after its operand's last use: no second set of registers
                        a[u] = k + 1 < NSB ? fetch(w[t & 1], k + 1, u) : fetch(w[(t + 1) & 1], 0, u);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                // the values are here: what they were read from may be overwritten
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) asm volatile("" : "+v"(xv[(t + 1) & 1][r][nt]));
                if (closes) asm volatile("" : "+v"(scales_next));
                request(s + 1 + D, t + 1 + D);
                if (closes) add_scaled(scales);
            }
        }
    }
    wait_requests<0>();                                 // those past the end: the LDS is used again

    // Sum over the wavefronts' K slices as in the centroid kernel.  Lane (i16, q): rows 8 i16 .. + 7, batch rows 16 nt + 4 q + e.
    typedef SliceSums<THREADS, BT, RB, KW> Sums;
    float* parts = reinterpret_cast<float*>(smem);
    __syncthreads();                                    // everyone is done with the table
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int b = 4 * q + e;
            if (b < BR && b0 + BR * nt + b < p.B) {
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = GS ? sum[GS ? nt : 0][GS ? u : 0][e] : acc[nt][u][e];
                float* dst = parts + (wave * BT + BR * nt + b) * Sums::kStride + i16 * 8;
                *reinterpret_cast<float4_t*>(dst) = float4_t{v[0], v[1], v[2], v[3]};
                *reinterpret_cast<float4_t*>(dst + 4) = float4_t{v[4], v[5], v[6], v[7]};
            }
        }
    Sums::finish(p, mm, parts, scale_bits, tid, blk, ks, b0);
}

template <int M, int V, int GS, int BR, int NT, int D>
int launch_gemm_staged_one(const Geometry& g, const GemmParams& p, hipStream_t stream)
{
    auto fn = gemm_staged_kernel<M, V, GS, BR, NT, D>;
    typedef StagedShape<M, V, GS, BR, NT, D> S;
    if (g.RB != kGranuleRows || g.BG != BR * NT) return CODEGEMM_UNSUPPORTED;
    constexpr size_t stage = SliceSums<S::kWaves * kWave, BR * NT, kGranuleRows, S::kWaves>::kLds;
    constexpr size_t lds = stage > S::kLds ? stage : S::kLds;
    static_assert(lds <= (size_t)kMaxLds, "LDS");
    int st = set_max_lds(reinterpret_cast<const void*>(fn), lds);
    if (st != CODEGEMM_OK) return st;
    const dim3 grid((unsigned)g.NKS, (unsigned)g.NBLK, (unsigned)g.NG);
    hipLaunchKernelGGL(fn, grid, dim3(S::kWaves * kWave), lds, stream, CG_HEAD_ARGS(p), p);
    return hipGetLastError() == hipSuccess ? CODEGEMM_OK : CODEGEMM_LAUNCH_FAILED;
}

// Two stages everywhere: three or four are no faster (v8 m2 g128, four rows, 8192->28672: 19.1, 19.5 us with four) and leave less
// room for batch rows.
template <int M, int V, int GS>
int launch_gemm_staged(const Geometry& g, const GemmParams& p, hipStream_t stream)
{
    constexpr bool WIDE = V == 8 && M == 1;
    switch (g.BG) {
        case 4:
            if constexpr (GS == 1) return launch_gemm_staged_one<M, V, GS, 4, 1, 2>(g, p, stream);
            break;
        case 8:
            if constexpr (GS == 1 && WIDE) return launch_gemm_staged_one<M, V, GS, 8, 1, 2>(g, p, stream);
            break;
        case 16:
            if constexpr (GS == 0 || !WIDE) return launch_gemm_staged_one<M, V, GS, 16, 1, 2>(g, p, stream);
            break;
        case 32:
            if constexpr (GS == 0 && !WIDE) return launch_gemm_staged_one<M, V, GS, 16, 2, 2>(g, p, stream);
            break;
    }
    return CODEGEMM_UNSUPPORTED;
}

}  // namespace cg
