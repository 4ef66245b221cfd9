// The 64x64 tile of the block-scaled FP4 GEMM: small problems, the leftover rectangles of a launch plan, and every shape
// that the larger tiles cannot take (any M and N, any K % 16 == 0).
//
// What bounds such a launch is latency: a few hundred workgroups, each with a long serial chain over K.  So the waves of
// a workgroup share the tile and cut K between them: each wave multiplies the whole 64x64 tile over every NW-th 128-k
// unit, copied into LDS stages of its own (no barriers; the next unit's copies are under way while one is multiplied),
// and the waves' partial tiles meet in LDS once, added in wave order.  A 64x64 wave tile expands four fragments for four
// matrix instructions (eight vector instructions each) where four 32x32 wave tiles of one workgroup expand eight, and
// the units that a workgroup has in flight at a time are neighbours in memory, so full cache lines are used.
// Measured (bf16 out, us; one 32x32 tile per wave over all of K before): 32x3072x3072 13.0 -> 9.0, 200x3072x3072
// 13.6 -> 10.3, 200x3072x14336 51.6 -> 29.9; 1000x3076x3088, which took a kernel of 128x128 tiles with f16 staged in LDS,
// 97 -> 38, 3520x3076x3088 208 -> 104 (640 TFLOP/s).  A unit takes about 0.25 us of a compute unit; its matrix
// instructions alone 0.15 and its expansions alone 0.18 (at the clock this load runs at), its copies alone 0.2.
// The exact route is that of nvfp4_gemm_tile.h: code x block scale is an exact f16 number, fp32 accumulation.
// The partial unit at the end of K is loaded in guarded 8-byte pieces, so nothing is read outside the operands.
#include "nvfp4_gemm_tile.h"

namespace nvfp4 {

typedef uint4v uint4v_a8 __attribute__((aligned(8)));          // an odd N leaves rows of a bf16 output on 8-byte boundaries
typedef uint2v uint2v_a1 __attribute__((aligned(1)));          // an odd K leaves rows of scales on any

constexpr int kSplitTile = 64, kSplitUnit = 128;
constexpr int kCodeBytes = 2 * kSplitTile * (kSplitUnit / 2), kStageBytes = kCodeBytes + 2 * kSplitTile * (kSplitUnit / 16);

template <int EPI_ACT, int NW, int STAGES, bool ODD>
__global__ __launch_bounds__(NW * 64, 2) void gemm_split_kernel(GemmArgs g)
{
    constexpr int EPI = EPI_ACT & 3;
    constexpr bool GELU = (EPI_ACT & kEpiGelu) != 0, LORA = (EPI_ACT & kEpiLora) != 0;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane & 31, lhalf = lane >> 5;
    const int64_t m0 = (int64_t)(blockIdx.x / g.n_tiles_n) * kSplitTile, n0 = (int64_t)(blockIdx.x % g.n_tiles_n) * kSplitTile;
    const int64_t kbytes = g.K >> 1, kblocks = g.K >> 4;
    const int full = (int)(g.K / kSplitUnit), rest = (int)(g.K % kSplitUnit);     // whole units, elements of the last one
    const int units = full + (rest != 0);
    const GemmEpilogue &ep = g.ep;
    // (read before anything else: behind the main loop each would be a trip to memory of its own)
    const float alpha = (*g.gsA) * (*g.gsW);
    const float sg_given = EPI == kEpiQuant ? *ep.q_scale : 0.0f;

    // ---- full units through LDS: copy instruction x of a unit fetches 16 rows, four lanes a row (a row-scattered load of
    // one row per lane costs about 60 cycles of the compute unit's address path per instruction; these a quarter), into
    // this wave's stage of the unit.  Staged rows 0-63: A, 64-127: W (rows past the end repeat the last one and are not
    // stored); 16-byte chunk c of staged row r sits in slot 4 r + (c ^ ((r >> 2) & 3)), as in the larger tiles.
    // Scales: eight bytes a row behind the codes, two lanes a row.  Rows of scales that do not start on dwords (ODD) cannot
    // be copied into LDS; they come into registers as eight bytes per lane, lane = row.
    typedef __attribute__((address_space(3))) void *lds_ptr_t;
    typedef const __attribute__((address_space(1))) void *global_ptr_t;
    uint8_t *const stage0 = lds + wave * (STAGES * kStageBytes);
    const uint8_t *cp[8], *sp[4];
#pragma unroll
    for (int x = 0; x < 8; ++x) {
        const int r = 16 * x + (lane >> 2), chunk = (lane & 3) ^ ((r >> 2) & 3);
        cp[x] = (x < 4 ? g.codesA + min(m0 + r, g.M - 1) * kbytes : g.codesW + min(n0 + (r - 64), g.N - 1) * kbytes) + 16 * chunk;
    }
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        const int r = ODD ? 64 * x + lane : 32 * x + (lane >> 1);
        const bool isA = ODD ? x == 0 : x < 2;
        if (!ODD || x < 2)
            sp[x] = (isA ? g.scalesA + min(m0 + r, g.M - 1) * kblocks : g.scalesW + min(n0 + (r - 64), g.N - 1) * kblocks) + (ODD ? 0 : 4 * (lane & 1));
    }
    uint2v sraw[STAGES][2];                        // ODD
    auto copy = [&](int u, auto stage_c) {
        constexpr int st = decltype(stage_c)::value;
#pragma unroll
        for (int x = 0; x < 8; ++x)
            __builtin_amdgcn_global_load_lds((global_ptr_t)(cp[x] + (int64_t)u * 64), (lds_ptr_t)(stage0 + st * kStageBytes + x * 1024), 16, 0, 0);
        if constexpr (ODD) {
#pragma unroll
            for (int x = 0; x < 2; ++x) sraw[st][x] = *(const uint2v_a1 *)(sp[x] + (int64_t)u * 8);
        } else {
#pragma unroll
            for (int x = 0; x < 4; ++x)
                __builtin_amdgcn_global_load_lds((global_ptr_t)(sp[x] + (int64_t)u * 8), (lds_ptr_t)(stage0 + st * kStageBytes + kCodeBytes + x * 256), 4, 0, 0);
        }
    };
    struct Unit {                                  // fragments 0, 1: A; 2, 3: W; lane = (row, half of the unit)
        uint4v c[4][2];
        uint32_t s[4];
    };
    auto read = [&](auto stage_c, Unit &x) {
        constexpr int st = decltype(stage_c)::value;
#pragma unroll
        for (int f = 0; f < 4; ++f)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                x.c[f][h] = *(const uint4v *)(stage0 + st * kStageBytes + (32 * f + lrow) * 64 + (((2 * lhalf + h) ^ ((lrow >> 2) & 3)) << 4));
        if constexpr (ODD) {
#pragma unroll
            for (int o = 0; o < 2; ++o) {          // rows 0-31 / 32-63: (low dword of the lower half, high dword of the upper half) each
                const auto p = __builtin_amdgcn_permlane32_swap(sraw[st][o].x, sraw[st][o].y, false, false);
                x.s[2 * o] = p[0];
                x.s[2 * o + 1] = p[1];
            }
        } else {
#pragma unroll
            for (int f = 0; f < 4; ++f)
                x.s[f] = *(const uint32_t *)(stage0 + st * kStageBytes + kCodeBytes + (32 * f + lrow) * 8 + 4 * lhalf);
        }
    };
    // the partial unit at the end of K, straight into registers in guarded pieces
    auto load_rest = [&](Unit &x) {
        const int blocks = min(max(rest / 16 - 4 * lhalf, 0), 4);          // this lane's blocks of it
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            const int64_t row = f < 2 ? min(m0 + 32 * f + lrow, g.M - 1) : min(n0 + 32 * (f - 2) + lrow, g.N - 1);
            const uint8_t *c = (f < 2 ? g.codesA : g.codesW) + row * kbytes + (int64_t)full * 64 + 32 * lhalf;
            const uint8_t *b8 = (f < 2 ? g.scalesA : g.scalesW) + row * kblocks + (int64_t)full * 8 + 4 * lhalf;
            uint2v p[4];
            uint32_t sc = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                p[b] = b < blocks ? *(const uint2v *)(c + 8 * b) : uint2v{0u, 0u};
                if (b < blocks) sc |= (uint32_t)b8[b] << (8 * b);
            }
            x.c[f][0] = uint4v{p[0].x, p[0].y, p[1].x, p[1].y};
            x.c[f][1] = uint4v{p[2].x, p[2].y, p[3].x, p[3].y};
            x.s[f] = sc;
        }
    };
    float16v acc[2][2];                                                    // [W fragment][A fragment]
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    auto multiply = [&](const Unit &x) {
        __builtin_amdgcn_sched_barrier(0);
        uint32_t sc[4][2];                                                 // a lane's four block scales as two pairs of f16
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            sc[f][0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(x.s[f], 1.0f, false));
            sc[f][1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(x.s[f], 1.0f, true));
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {                                      // eight codes of every lane: sixteen k
            half8v frag[4];
#pragma unroll
            for (int f = 0; f < 4; ++f) {
                const uint32_t w = x.c[f][q >> 2][q & 3];
                const half2v pair = __builtin_bit_cast(half2v, sc[f][q >> 2]);
                const half2v p = (q & 2) ? half2v{pair.y, pair.y} : half2v{pair.x, pair.x};
                uint4v o;
                o.x = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 1.0f, 0) * p);
                o.y = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 1.0f, 1) * p);
                o.z = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 1.0f, 2) * p);
                o.w = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 1.0f, 3) * p);
                frag[f] = __builtin_bit_cast(half8v, o);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(frag[2 + i], frag[j], acc[i][j], 0, 0, 0);
        }
        // the expansions of the next sixteen k issue in the shadow of the matrix instructions: eight behind each
        __builtin_amdgcn_sched_group_barrier(0x2, 40, 0);
#pragma unroll
        for (int k = 0; k < 32; ++k) {
            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x2, 8, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // ---- this wave's units: wave, wave + NW, ...; the partial one, if any, while the first copies are under way
    static_for<0, STAGES>([&](auto st) {
        if (wave + decltype(st)::value * NW < full) copy(wave + decltype(st)::value * NW, st);
    });
    if constexpr (LORA) {
        // the low-rank update T B^T, on the wave whose turn the next unit would be, scaled so that the epilogue's one
        // multiplication by alpha leaves lora_scale T B^T (rank 128: sixteen consecutive k per matrix instruction)
        if (units % NW == wave) {
            typedef __bf16 bf16x8v __attribute__((ext_vector_type(8)));
            const uint16_t *lp[4];
#pragma unroll
            for (int f = 0; f < 4; ++f)
                lp[f] = (f < 2 ? g.lora_t + min(m0 + 32 * f + lrow, g.M - 1) * kLoraRank : g.lora_b + min(n0 + 32 * (f - 2) + lrow, g.N - 1) * kLoraRank) + 8 * lhalf;
#pragma unroll
            for (int k = 0; k < kLoraRank / 16; ++k) {
                uint4v v[4];
#pragma unroll
                for (int f = 0; f < 4; ++f) v[f] = *(const uint4v *)(lp[f] + 16 * k);
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8v, v[2 + i]), __builtin_bit_cast(bf16x8v, v[j]), acc[i][j], 0, 0, 0);
            }
            const float rescale = g.lora_scale / alpha;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[i][j][r] *= rescale;
        }
    }
    if (rest != 0 && full % NW == wave) {
        Unit x;
        load_rest(x);
        multiply(x);
    }
    for (int u0 = wave; u0 < full; u0 += STAGES * NW) {
        static_for<0, STAGES>([&](auto st) {
            const int u = u0 + decltype(st)::value * NW;
            if (u >= full) return;
            // the copies of this unit have landed when at most those of the later ones in flight are outstanding
            if (u + (STAGES - 1) * NW < full) wait_vmcnt_le<(STAGES - 1) * (ODD ? 10 : 12)>();
            else wait_vmcnt_le<0>();
            NVFP4_COMPILER_FENCE();
            Unit x;
            read(st, x);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");             // the stage has been read: it may be filled again
            if (u + STAGES * NW < full) copy(u + STAGES * NW, st);
            multiply(x);
        });
    }
    __syncthreads();                                // (the stages become the slabs of the partial tiles)

    // ---- the waves' partial tiles meet in LDS.  After the matrix instructions a lane holds row lrow of an A fragment and,
    // in register 4 q + e, column 8 q + 4 lhalf + e of a W fragment: four consecutive columns per 16-byte granule.
    // Granule (row, c4 = column / 4) of wave w lies at  w * 16 KB + c4 * 1 KB + (row with its low bits XOR c4) * 16 B:
    // what a wave writes at a time (32 rows of one c4) and what sixteen lanes read at a time (one row) fall on distinct banks.
    const int used = min(NW, units + (LORA ? 1 : 0));
    float4v *slab = (float4v *)lds;
    if (wave < used) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int c4 = 8 * i + 2 * q + lhalf;
                    slab[wave * 1024 + c4 * 64 + ((32 * j + lrow) ^ c4)] =
                        float4v{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
                }
    }
    __syncthreads();
    TensorScale ts{};
    if constexpr (EPI == kEpiQuant) {
        if (blockIdx.x == 0 && tid == 0) *ep.q_scale_out = sg_given;
        ts = tensor_scale(sg_given);
    }
    uint32_t hmax = 0;                                                     // largest |bf16| pattern seen by this lane
    // a thread finishes items of W consecutive columns of one row (16 bytes of output, or one block to re-quantize)
    constexpr int W = EPI == kEpiF32 ? 4 : (EPI == kEpiBF16 ? 8 : 16), PER_ROW = kSplitTile / W;
    for (int t = tid; t < kSplitTile * PER_ROW; t += NW * 64) {
        const int r = t / PER_ROW, c = t % PER_ROW;
        const int64_t m = m0 + r, n = n0 + c * W;
        if (m >= g.M || n >= g.N) continue;
        float y[W];
#pragma unroll
        for (int v = 0; v < W / 4; ++v) {
            const int c4 = c * (W / 4) + v, at = c4 * 64 + (r ^ c4);
            float4v sum = slab[at];
            for (int w = 1; w < used; ++w) sum += slab[w * 1024 + at];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float o = sum[e] * alpha;
                if constexpr (GELU) o = gelu_tanh_f32(o);
                y[4 * v + e] = o;
            }
        }
        if constexpr (EPI == kEpiF32) {
            float *dst = (float *)ep.Y + m * ep.ldy + n;
            const float4v o = {y[0], y[1], y[2], y[3]};
            if (n + W <= g.N) {
                if (ep.stream_out) __builtin_nontemporal_store(o, (float4v *)dst);
                else *(float4v *)dst = o;
            } else {
                for (int e = 0; e < W && n + e < g.N; ++e) dst[e] = y[e];
            }
        } else {
            uint32_t h[W / 2];
#pragma unroll
            for (int v = 0; v < W / 2; ++v) {
                h[v] = pack_bf16x2(y[2 * v], y[2 * v + 1]);
                if (ep.amax_partial) hmax = pk_absmax_u16(hmax, h[v]);      // (columns past the end repeat the last one)
            }
            if (EPI == kEpiBF16 || ep.Y != nullptr) {
                uint16_t *dst = (uint16_t *)ep.Y + m * ep.ldy + n;
                if (n + W <= g.N) {
#pragma unroll
                    for (int v = 0; v < W / 8; ++v) {
                        const uint4v o = {h[4 * v], h[4 * v + 1], h[4 * v + 2], h[4 * v + 3]};
                        if (ep.stream_out) __builtin_nontemporal_store(o, (uint4v_a8 *)(dst + 8 * v));
                        else *(uint4v_a8 *)(dst + 8 * v) = o;
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < W; ++e)
                        if (n + e < g.N) dst[e] = (uint16_t)(h[e >> 1] >> (16 * (e & 1)));
                }
            }
            if constexpr (EPI == kEpiQuant) {                              // N % 16 == 0: a block is all in or all out
                if (__builtin_expect(ts.shift != 1.0f, 0)) rescale_block16(h, ts.shift);
                uint32_t sbyte, c0, c1;
                quantize_block16(h, ts, sbyte, c0, c1);
                *(uint2v *)(ep.q_codes + m * (g.q_pitch >> 1) + (n >> 1)) = uint2v{c0, c1};
                ep.q_scales[m * (g.q_pitch >> 4) + (n >> 4)] = (uint8_t)sbyte;
            }
        }
    }
    if (ep.amax_partial) {
        uint32_t *wmax = (uint32_t *)(lds + NW * max(STAGES * kStageBytes, 16384));
        const uint32_t mx = wave_max_u32(pk_hmax_u16(hmax));
        if (lane == 0) wmax[wave] = mx;
        __syncthreads();
        if (tid == 0) {
            uint32_t all = wmax[0];
#pragma unroll
            for (int w = 1; w < NW; ++w) all = max(all, wmax[w]);
            ep.amax_partial[g.partial_base + blockIdx.x] = all;
        }
    }
}

template <int EPI, int NW, int STAGES, bool ODD>
static hipError_t launch_split(const GemmArgs &g, int64_t tiles, hipStream_t s)
{
    constexpr int smem = NW * std::max(STAGES * kStageBytes, 16384) + 64;
    static uint64_t attr_set = 0;          // the dynamic LDS limit is raised once per kernel variant and device
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev); e != hipSuccess) return e;
    if (((attr_set >> (dev & 63)) & 1u) == 0) {
        hipError_t e = hipFuncSetAttribute((const void *)gemm_split_kernel<EPI, NW, STAGES, ODD>, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
        if (e != hipSuccess) return e;
        attr_set |= 1ull << (dev & 63);
    }
    GemmArgs a = g;
    a.n_tiles_n = (int)((g.N + kSplitTile - 1) / kSplitTile);
    gemm_split_kernel<EPI, NW, STAGES, ODD><<<(unsigned)tiles, NW * 64, smem, s>>>(a);
    return hipGetLastError();
}

template <int NW, int STAGES>
static hipError_t launch_split_epi(int epi, const GemmArgs &g, int64_t tiles, hipStream_t s)
{
    const bool odd = (g.K & 63) != 0;              // rows of scales off the dword grid
    switch (epi) {
    case kEpiF32: return odd ? launch_split<kEpiF32, NW, STAGES, true>(g, tiles, s) : launch_split<kEpiF32, NW, STAGES, false>(g, tiles, s);
    case kEpiBF16: return odd ? launch_split<kEpiBF16, NW, STAGES, true>(g, tiles, s) : launch_split<kEpiBF16, NW, STAGES, false>(g, tiles, s);
    case kEpiBF16 | kEpiGelu:
        return odd ? launch_split<kEpiBF16 | kEpiGelu, NW, STAGES, true>(g, tiles, s) : launch_split<kEpiBF16 | kEpiGelu, NW, STAGES, false>(g, tiles, s);
    // (re-quantizing epilogues: planned problems only, K % 64 == 0)
    case kEpiQuant: return odd ? hipErrorInvalidValue : launch_split<kEpiQuant, NW, STAGES, false>(g, tiles, s);
    case kEpiQuant | kEpiGelu: return odd ? hipErrorInvalidValue : launch_split<kEpiQuant | kEpiGelu, NW, STAGES, false>(g, tiles, s);
    // (planned problems only as well)
    case kEpiF32 | kEpiLora: return odd ? hipErrorInvalidValue : launch_split<kEpiF32 | kEpiLora, NW, STAGES, false>(g, tiles, s);
    case kEpiBF16 | kEpiLora: return odd ? hipErrorInvalidValue : launch_split<kEpiBF16 | kEpiLora, NW, STAGES, false>(g, tiles, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_tile_64x64(int epi, const GemmArgs &g, int64_t tiles, hipStream_t s)
{
    // Up to four units only as many waves have work, and the other four help to finish the tile (256x1536x512: 4.4 us
    // against 4.7); beyond, four waves and two workgroups to a compute unit (3520x3076x3088: 104 us against 129).
    return g.K <= 4 * kSplitUnit ? launch_split_epi<8, 2>(epi, g, tiles, s) : launch_split_epi<4, 2>(epi, g, tiles, s);
}

}  // namespace nvfp4
