// The centroid kernel for prompts: more than 32 batch rows, fp16 output (fp32 output needs sums that there are no registers
// for here, and a spread of K over wavefronts: the centroid kernel's tiles along the grid).  Included by gemm_centroid_m1.hip ..
// gemm_centroid_m4.hip; mapping, table, lookups and the kinds of scales (GS) as in gemm_centroid_impl.h.
//
// A lookup is paid once per 64 codes whatever the batch, so with NT tiles of 16 batch rows per
// wavefront the matrix cores take over as the bound (NT = 4: 32 lookups, 64 for v = 4, and 128 MFMAs
// per step and codebook; counters at 8192^2 v8 m2 batch 2048: matrix cores 85 % busy, LDS 29 %), at the clock
// that their power leaves: 1.87 GHz there, 2.37 with x = 0.  Each of the 8 wavefronts owns 128 rows and streams
// through the whole of K, there is nothing to sum across wavefronts or workgroups, and x is staged in LDS for all of
// them: one step (16 chunks of 16 bytes, 128 elements) of 16 NT batch rows, double-buffered, one barrier per step.
// Measured in one run: 8192^2 v8 m2 at batch 2048 375 us (357 on other boxes), 281 with x = 0, 64 launches of 32 rows 1231.
// The two codebooks make it 550 GFLOP of MFMAs: 1.47 to 1.54 PFLOP/s; this instruction alone, in registers, reaches 1.87.
//
// UR: rows of an octet that a wavefront takes, 8 or (v4 m1 with group scales) 4.  With sums of their own beside the accumulators there are
// registers for two tiles of 8 rows, and then v = 4, which needs two lookups per MFMA operand, is bound by the LDS (4.5 cycles per
// MFMA and compute unit, an MFMA takes 4).  Four tiles of 4 rows hold as many sums and make it 3: two neighbouring wavefronts share a
// granule, each with its half of every octet.  4096->28672 v4 m1 g128, batch 500: 129 -> 123 us, g32 159 -> 148.  Where it makes one more round
// of workgroups UR stays 8 (make_geometry).
//
// Chunk 4 q + j of row r lies at place (4 j + q) ^ (r % 16) of its 256-byte row: the operand reads of a round take lanes of all four q
// in one LDS cycle, and with the chunks in order (place (4 q + j) ^ (r % 16)) these were 2-way conflicts (3.5 against 1.9 ns per read).
// Group scales go onto the sums of row u - 1 beside the MFMAs of row u, and the codes of the next step are put in order at the end
// of the step before it, a step after they were asked for.
#pragma once

#include "gemm_centroid_impl.h"
#include "gemm_staged_impl.h"

namespace cg {

typedef uint32_t u32x3_t __attribute__((ext_vector_type(3)));

template <int M, int V, int NT, int GS, int UR>
__global__ void __launch_bounds__(512) gemm_prompt_kernel(CG_HEAD_PARAMS, const GemmParams pk)
{
    const GemmParams p = with_head(pk, hx, hpacked, hcodebooks, hgscales, hK, hNKT, hKPW, hB, hNGR, hmisc);
    typedef CentroidTable<M, V> T;
    static_assert(V == 4 || V == 8, "a step is 128 elements of x");
    constexpr int NW = 8;
    constexpr int THREADS = NW * kWave;
    constexpr int SPU = V == 4 ? 1 : 2;                // steps per unit of 32 sub-vectors
    constexpr int NSB = 4 * M;                         // (round, codebook) per step
    constexpr int PW = V == 4 ? 8 : 4;                 // dwords per lane and round of a part with two codebooks
    constexpr bool HALF = UR == 4;                     // a wavefront takes 4 rows of each octet, its neighbour the other 4
    static_assert(UR == 8 || (V == 4 && M == 1), "8 rows per lane");
    constexpr int WR = HALF ? 2 : PW / 2 * M;          // dwords of codes per lane and round
    constexpr int BT = 16 * NT;                        // batch rows of the workgroup
    constexpr int XL = BT * 16 / THREADS;              // chunks of x this thread moves per step
    constexpr int kUnitBytes = kGranuleRows * kSlots * M;
    constexpr bool SCALED = GS != 0;
    constexpr int kOutOfRange = 0x7ffffff0;
    constexpr uint32_t kRsrcFlags = 0x00020000u;
    static_assert(BT * 16 % THREADS == 0, "whole chunks per thread");

    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const Member& mm = p.mem[0];
    const int gr = HALF ? blockIdx.x * (NW / 2) + wave / 2 : blockIdx.x * NW + wave;       // the wavefront's granule
    const int half = HALF ? wave & 1 : 0;
    const int b0 = blockIdx.y * BT;
    const int steps = p.NKT * SPU;
    const int q = lane >> 4, i16 = lane & 15, lo = i16 >> 1;
    const bool odd = lane & 1;

    // table entries, requested first
    constexpr int ENTRIES = M * kCentroids;
    constexpr int TPE = 2 * ENTRIES <= THREADS ? 2 : 1;
    constexpr int EPT = (ENTRIES + THREADS - 1) / THREADS;
    typedef typename Frag<V == 4 ? 4 : 16>::type entry_t;
    entry_t fill[EPT];
#pragma unroll
    for (int k = 0; k < EPT; ++k) fill[k] = reinterpret_cast<const entry_t*>(mm.codebooks)[TPE > 1 ? min(tid / TPE, ENTRIES - 1) : min(tid + k * THREADS, ENTRIES - 1)];

    // x: thread -> chunk tid % 16 of row tid / 16 (+ 32)
    const __amdgpu_buffer_rsrc_t x_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<_Float16*>(p.x + (size_t)b0 * p.K), 0, min(p.B - b0, BT) * p.K * 2, kRsrcFlags);
    const int xc = tid & 15, xrow = tid >> 4;
    const int place = GS == 2 ? xc : 4 * (xc & 3) + (xc >> 2);           // 4 j + q of the lanes that read chunk xc
    const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>((lds_float*)smem);
    const uint32_t xbase = lds0 + (uint32_t)T::kBytes;
    u32x4_t xl[XL];
    auto load_x = [&](int s) {
        const int el = s * 128 + xc * 8;
#pragma unroll
        for (int k = 0; k < XL; ++k)
            xl[k] = __builtin_amdgcn_raw_buffer_load_b128(x_rsrc, el < p.K ? ((xrow + 32 * k) * p.K + el) * 2 : kOutOfRange, 0, 0);
    };
    auto store_x = [&](int s) {
        const bool past = V == 4 && s * 128 + xc * 8 + 4 >= p.K;        // an odd number of sub-vectors: the chunk reaches past the row
#pragma unroll
        for (int k = 0; k < XL; ++k) {
            u32x4_t t = xl[k];
            if constexpr (V == 4) {
                t.z = past ? 0u : t.z;
                t.w = past ? 0u : t.w;
            }
            const uint32_t a = xbase + (uint32_t)((s & 1) * (BT * 256) + (xrow + 32 * k) * 256 + ((place ^ (xrow & 15)) * 16));
            *reinterpret_cast<lds_half8*>(static_cast<uintptr_t>(a)) = __builtin_bit_cast(half8_t, t);
        }
    };
    // codes of a step, pairs of loads with pairs of lanes along memory
    const uint8_t* cbase = mm.packed + (size_t)min(gr, mm.NGR - 1) * p.NKT * kUnitBytes;
    const __amdgpu_buffer_rsrc_t c_rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(cbase), 0, gr < mm.NGR ? p.NKT * kUnitBytes : 0, kRsrcFlags);
    // chunk of load j: GS = 2 as in the centroid kernel, every MFMA contracting over 4 neighbouring chunks
    const int c_ent = 2 * lo * kSlots + (V == 4 ? 2 : 1) * ((GS == 2 ? 4 * (q & 1) + 2 * (q >> 1) : 4 * q) + (lane & 1));
    auto load_codes = [&](uint32_t (&dst)[4][WR], int s) {
        const int unit = (s / SPU) * kUnitBytes;       // past the last unit: zeros
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int ent = c_ent + (V == 4 ? 0 : (s % SPU) * 16) + (V == 4 ? 2 : 1) * ((GS == 2 ? 8 : 2) * (j / 2)) + (j % 2) * kSlots;
#pragma unroll
            for (int part = 0; part < (M + 1) / 2; ++part) {
                uint32_t* w = dst[j] + part * PW;
                if (2 * part + 1 == M) {
                    if constexpr (V == 4) {
                        if constexpr (HALF) {          // rows 4 half .. + 3 of two sub-vectors, and what lies between
                            const u32x3_t t = __builtin_amdgcn_raw_buffer_load_b96(c_rsrc, unit + ent * 8 + 4 * half, 0, 0);
                            w[0] = t.x; w[1] = t.z;
                            continue;
                        }
                        const u32x4_t t = __builtin_amdgcn_raw_buffer_load_b128(c_rsrc, unit + part * 8192 + ent * 8, 0, 0);
                        w[0] = t.x; w[1] = t.y; w[2] = t.z; w[3] = t.w;
                    } else {
                        const u32x2_t t = __builtin_amdgcn_raw_buffer_load_b64(c_rsrc, unit + part * 8192 + ent * 8, 0, 0);
                        w[0] = t.x; w[1] = t.y;
                    }
                } else {
#pragma unroll
                    for (int g = 0; g < PW / 4; ++g) {
                        const u32x4_t t = __builtin_amdgcn_raw_buffer_load_b128(c_rsrc, unit + part * 8192 + (ent + g) * 16, 0, 0);
                        w[4 * g] = t.x; w[4 * g + 1] = t.y; w[4 * g + 2] = t.z; w[4 * g + 3] = t.w;
                    }
                }
            }
        }
    };
    const int order = T::kOrderBits == 1 ? (lane >> 3) & 1 : 0;
    auto turn_codes = [&](uint32_t (&cw)[4][WR]) {
#pragma unroll
        for (int j = 0; j < 4; j += 2)
#pragma unroll
            for (int k = 0; k < WR; ++k) {
                pair_transpose(cw[j][k], cw[j + 1][k], odd);
                if constexpr (GS == 2) row_exchange(cw[j][k], cw[j + 1][k]);
            }
        if constexpr (T::kOrderBits == 1) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int part = 0; part < M / 2; ++part)
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        uint32_t* w = cw[j] + part * PW;
                        const uint32_t a = w[k], b = w[2 + k];
                        w[k] = order ? b : a;
                        w[2 + k] = order ? a : b;
                    }
        }
    };
    __amdgpu_buffer_rsrc_t s_rsrc;
    if constexpr (SCALED) {
        const uint8_t* base = mm.gscales + (size_t)min(gr, mm.NGR - 1) * p.NKT * p.GPU * 256;
        s_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(base), 0, gr < mm.NGR ? p.NKT * p.GPU * 256 : 0, kRsrcFlags);
    }
    constexpr int SR = GS == 2 ? 4 : 1;                // scales per step
    auto load_scales = [&](half8_t (&dst)[SR], int s) {
#pragma unroll
        for (int j = 0; j < SR; ++j) {
            const int sub = (s % SPU) * 16 + (V == 4 ? 2 : 1) * 4 * j;  // of the unit
            const int o = ((s / SPU) * p.GPU + (sub >> p.gshift)) * 256;
            if constexpr (HALF) {
                const half4_t t = __builtin_bit_cast(half4_t, __builtin_amdgcn_raw_buffer_load_b64(s_rsrc, o + i16 * 16 + 8 * half, 0, 0));
                dst[j] = __builtin_shufflevector(t, t, 0, 1, 2, 3, 0, 1, 2, 3);
            } else {
                dst[j] = __builtin_bit_cast(half8_t, __builtin_amdgcn_raw_buffer_load_b128(s_rsrc, o + i16 * 16, 0, 0));
            }
        }
    };

    uint32_t w[2][4][WR];
    half8_t sc[2][SR];
    __builtin_amdgcn_sched_barrier(0);
    load_x(0);
    load_codes(w[0], 0);
    if constexpr (SCALED) load_scales(sc[0], 0);
    load_codes(w[1], 1);
    if constexpr (SCALED) load_scales(sc[1], 1);
    __builtin_amdgcn_sched_barrier(0);

#pragma unroll
    for (int k = 0; k < EPT; ++k) {
        const int e = TPE > 1 ? tid / TPE : tid + k * THREADS;
        if (e < ENTRIES) {
            const int code = e % kCentroids, c = e / kCentroids;
            const uint32_t row = lds0 + (uint32_t)(T::plane(c, 0) * 65536 + code * 256 + T::region(c));
            const int cols = T::columns(c), mine = cols / TPE;
            const int c0 = (TPE > 1 ? (tid % TPE) * mine + tid / TPE : lane);
            for (int j = 0; j < mine; ++j) {
                const uint32_t a = row + (uint32_t)((c0 + j) & (cols - 1)) * T::kEntry;
                if constexpr (V == 4) *reinterpret_cast<lds_half4*>(static_cast<uintptr_t>(a)) = fill[k];
                else *reinterpret_cast<lds_half8*>(static_cast<uintptr_t>(a)) = fill[k];
            }
        }
    }
    store_x(0);
    load_x(1);

    float4_t acc[NT][UR];
    float4_t sum[GS ? NT : 1][GS ? UR : 1];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int u = 0; u < UR; ++u) {
            acc[nt][u] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
            if constexpr (GS) sum[nt][u] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
        }

    uint32_t base[M];
#pragma unroll
    for (int k = 0; k < M; ++k) {
        const bool alone = k == M - 1 && (M & 1);
        const int c = alone ? k : k ^ order;
        base[k] = lds0 + (uint32_t)((alone ? T::region(k) : T::kOrderBits == 1 ? (c % 2) * T::region(1) : T::region(k)) +
                                    (lane & (T::columns(k) - 1)) * T::kEntry) + (uint32_t)(T::plane(k, 0) << 16);
    }
    auto fetch = [&](const uint32_t (&cw)[4][WR], int k, int u) -> half8_t {
        const int c = k % M, j = k / M;
        const uint32_t* wj = cw[j] + (c / 2) * PW;
        const bool single = 2 * (c / 2) + 1 == M;
        const uint32_t sel = 0x0c020000u | (uint32_t)(4 + u % 4) << 8;
        const uint32_t w0 = HALF ? wj[0] : single ? wj[u / 4] : wj[2 * (c % 2) + u / 4];
        if constexpr (V == 4) {
            const uint32_t w1 = HALF ? wj[1] : single ? wj[2 + u / 4] : wj[4 + 2 * (c % 2) + u / 4];
            const half4_t lo4 = *reinterpret_cast<const lds_half4*>(static_cast<uintptr_t>(__builtin_amdgcn_perm(w0, base[c], sel)));
            const half4_t hi4 = *reinterpret_cast<const lds_half4*>(static_cast<uintptr_t>(__builtin_amdgcn_perm(w1, base[c], sel)));
            return __builtin_shufflevector(lo4, hi4, 0, 1, 2, 3, 4, 5, 6, 7);
        } else {
            return *reinterpret_cast<const lds_half8*>(static_cast<uintptr_t>(__builtin_amdgcn_perm(w0, base[c], sel)));
        }
    };
    // Beside MFMAs, and the next codes turned late, but for v4 m2 with short groups, where both spill (2048->8192 g32, batch 512: 100
    // us, 90 with the sums behind the MFMAs and the codes turned first).  Other formats, time of that order / time here on random sizes: 1.00
    // to 1.11 for v8 m1, m2 and v4 m1, v4 m2 1.20, v8 m3 1.06, m4 1.39 with long and 1.05 with short groups, though these spill more (112 registers, 93).
    constexpr bool BESIDE = !(V == 4 && M == 2 && GS == 2);
    auto add_scaled = [&](const half8_t& scales, int u) {
        const float f = (float)scales[u];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[GS ? nt : 0][GS ? u : 0][e] = __builtin_fmaf(f, acc[nt][u][e], sum[GS ? nt : 0][GS ? u : 0][e]);
    };
    // x operand of (tile nt, round j): chunk 4 q + j (GS = 2: 4 j + q) of batch row 16 nt + i16
    const uint32_t xrd = xbase + (uint32_t)(i16 * 256);
    auto x_operand = [&](int s, int nt, int j) -> half8_t {
        return *reinterpret_cast<const lds_half8*>(static_cast<uintptr_t>(xrd + (uint32_t)((s & 1) * (BT * 256) + nt * 4096) + (uint32_t)(((4 * j + q) ^ i16) * 16)));
    };

    __syncthreads();

    half8_t a[UR], xv[NT];
    turn_codes(w[0]);
#pragma unroll
    for (int u = 0; u < UR; ++u) a[u] = fetch(w[0], 0, u);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) xv[nt] = x_operand(0, nt, 0);
    for (int s0 = 0; s0 < steps; s0 += 2) {
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const int s = s0 + d;                      // (an odd number of steps ends with one whose codes and x are zero)
            store_x(s + 1);
            load_x(s + 2);
            if constexpr (!BESIDE) turn_codes(w[d ^ 1]);
            if (s < steps) {
#pragma unroll
                for (int k = 0; k < NSB; ++k) {
                    const int j = k / M;
                    const bool closes = (GS == 1 && k == NSB - 1) || (GS == 2 && k % M == M - 1);      // a chain of sums
                    if (BESIDE && k == NSB - 1) turn_codes(w[d ^ 1]);  // asked for a step ago
#pragma unroll
                    for (int u = 0; u < UR; ++u) {
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) {
                            acc[nt][u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xv[nt], a[u], (GS == 1 && k == 0) || (GS == 2 && k % M == 0) ? float4_t{} : acc[nt][u], 0, 0, 0);
                        }
                        __builtin_amdgcn_sched_barrier(0);         // the lookup after its operand's last use: no second set of registers
                        a[u] = k + 1 < NSB ? fetch(w[d], k + 1, u) : fetch(w[d ^ 1], 0, u);
                        if (BESIDE && closes && u > 0) add_scaled(sc[d][GS == 2 ? j : 0], u - 1);    // beside the MFMAs of row u
                    }
                    if (k % M == M - 1 && j < 3) {
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) xv[nt] = x_operand(s, nt, j + 1);
                    }
                    if (closes) {
#pragma unroll
                        for (int u = BESIDE ? UR - 1 : 0; u < UR; ++u) add_scaled(sc[d][GS == 2 ? j : 0], u);
                    }
                }
            }
            load_codes(w[d], s + 2);
            if constexpr (SCALED) load_scales(sc[d], s + 2);
            __syncthreads();
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) xv[nt] = x_operand(s + 1, nt, 0);
        }
    }

    // Lane (i16, q): rows 8 i16 .. + 7 of the granule, batch rows 16 nt + 4 q + e.
    const int n0 = gr * kGranuleRows + i16 * kRowsPerLane + 4 * half;
    float scale[UR];
    if constexpr (SCALED) {
#pragma unroll
        for (int u = 0; u < UR; ++u) scale[u] = 1.0f;
    } else {
        const __amdgpu_buffer_rsrc_t r_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(mm.scales), 0, mm.N * 2, kRsrcFlags);
#pragma unroll
        for (int u = 0; u < UR; ++u)
            scale[u] = (float)__builtin_bit_cast(_Float16, __builtin_amdgcn_raw_buffer_load_b16(r_rsrc, (n0 + u) * 2, 0, 0));
    }
    const bool whole = n0 + UR <= mm.N;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int b = b0 + 16 * nt + 4 * q + e;
            if (b >= p.B || n0 >= mm.N) continue;
            float v[UR];
#pragma unroll
            for (int u = 0; u < UR; ++u) {
                v[u] = (GS ? sum[GS ? nt : 0][GS ? u : 0][e] : acc[nt][u][e]) * scale[u];
                asm volatile("" : "+v"(v[u]));         // an fp32 product, as in the other kernels: the compiler would round it to fp16 at once
            }
            _Float16* y = static_cast<_Float16*>(mm.y) + (size_t)b * mm.N + n0;
            if (whole && mm.N % UR == 0) {            // 16-byte stores need every row of y aligned
                typename Frag<HALF ? 4 : 16>::type h;      // 4 or 8 values
#pragma unroll
                for (int u = 0; u < UR; ++u) h[u] = (_Float16)v[u];
                *reinterpret_cast<decltype(h)*>(y) = h;
            } else {
#pragma unroll
                for (int u = 0; u < UR; ++u)
                    if (n0 + u < mm.N) y[u] = (_Float16)v[u];
            }
        }
}

template <int M, int V, int NT, int GS, int UR>
int launch_gemm_prompt_one(const Geometry& g, const GemmParams& p, hipStream_t stream)
{
    auto fn = gemm_prompt_kernel<M, V, NT, GS, UR>;
    constexpr size_t lds = CentroidTable<M, V>::kBytes + 2 * 16 * NT * 256;
    static_assert(lds <= (size_t)kMaxLds, "LDS");
    int st = set_max_lds(reinterpret_cast<const void*>(fn), lds);
    if (st != CODEGEMM_OK) return st;
    const dim3 grid((unsigned)ceil_div(g.NGR, UR), (unsigned)ceil_div(p.B, 16 * NT));
    hipLaunchKernelGGL(fn, grid, dim3(512), lds, stream, CG_HEAD_ARGS(p), p);
    return hipGetLastError() == hipSuccess ? CODEGEMM_OK : CODEGEMM_LAUNCH_FAILED;
}

template <int M, int V, int GS>
int launch_gemm_centroid_mv(const Geometry& g, const GemmParams& p, hipStream_t stream)
{
    if constexpr (V < 16 && GS <= 2) {
        if (g.prompt) {
            if constexpr (V == 4 && M == 1 && GS != 0) {
                if (g.half) return launch_gemm_prompt_one<M, V, 4, GS, 4>(g, p, stream);
            }
            return launch_gemm_prompt_one<M, V, prompt_tiles(M, V, GS != 0), GS, 8>(g, p, stream);
        }
    }
    if constexpr (GS <= 2 && ((V == 8 && M <= 2) || (V == 4 && M == 1))) {
        if (g.staged) return launch_gemm_staged<M, V, GS>(g, p, stream);
    }
    return launch_gemm_centroid_v<M, V, GS>(g, p, stream);
}

template <int M, int V>
int launch_gemm_centroid_mg(const Geometry& g, const GemmParams& p, hipStream_t stream)
{
    if (p.y_fp32) return g.g < 0 ? launch_gemm_centroid_mv<M, V, 3>(g, p, stream) : launch_gemm_centroid_mv<M, V, 4>(g, p, stream);
    if (g.g < 0) return launch_gemm_centroid_mv<M, V, 0>(g, p, stream);
    // a step, 16 chunks, is 16 sub-vectors (32 for v = 4)
    if (g.gshift >= (V == 4 ? 5 : 4)) return launch_gemm_centroid_mv<M, V, 1>(g, p, stream);
    return launch_gemm_centroid_mv<M, V, 2>(g, p, stream);
}

template <int M>
int launch_gemm_centroid_m(const Geometry& g, const GemmParams& p, hipStream_t stream)
{
    if (g.v == 16) return launch_gemm_centroid_mg<M, 16>(g, p, stream);
    if (g.v == 8) return launch_gemm_centroid_mg<M, 8>(g, p, stream);
    if constexpr (M <= 2) return launch_gemm_centroid_mg<M, 4>(g, p, stream);
    return CODEGEMM_UNSUPPORTED;
}

}  // namespace cg
