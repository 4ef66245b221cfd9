// Block-scaled FP4 GEMM for gfx950 (Sec. 2.2 / 3.1; Appendix "Implementation Details"): the host
// side (launch plan, chunking, dispatch to the tile shapes of nvfp4_gemm_tile.h and
// nvfp4_gemm_split.hip), and the down projection of the LoRA side branch.
#include "nvfp4_gemm_tile.h"
#include "nvfp4_gemm_plan.h"

namespace nvfp4 {

// ============================================================================
// Down projection of the LoRA side branch: T [M, 128] = bf16(X A^T), X [M, K] and A [128, K]
// bf16, fp32 accumulation on v_mfma_f32_32x32x16_bf16.  A skinny GEMM, bound by latency and by what a compute unit
// pulls: with whole-K tiles either few workgroups run or every one of them pulls all of A.  So K is cut:
// workgroup (i, s) multiplies rows 128 i .. 128 i + 127 with K range s of `splits` (2 x 2 waves of 64 x 64), writes
// an fp32 partial tile to the workspace, and a second small kernel adds the partial tiles in split order and rounds to
// bf16.  The 64-k steps of a range are copied straight into a ring of four LDS stages, so that most of a range (six steps
// of the 3520x3072 projection) is under way at once: 17.7 us for that
// projection, both kernels, with one step at a time through registers; 14.7 now (128x3072: 12.2 -> 7.7).
// ============================================================================
constexpr int kLdRows = 128;                                      // rows of X per workgroup
constexpr int kLdStages = 4, kLdStageBytes = (kLdRows + kLoraRank) * ROW_BYTES;      // 32 KB
static __device__ __align__(16) uint8_t g_zeros[16];              // what chunks past the end of K are copied from
__global__ __launch_bounds__(256) void lora_down_partial_kernel(const uint16_t *__restrict__ x, int64_t M,
                                                                int64_t K, int64_t ldx,
                                                                const uint16_t *__restrict__ a, int steps_per_split,
                                                                float *__restrict__ partial, int64_t m_pad)
{
#if defined(__HIP_DEVICE_COMPILE__)
    typedef __bf16 bf16x8v __attribute__((ext_vector_type(8)));
    typedef __attribute__((address_space(3))) void *lds_ptr_t;
    typedef const __attribute__((address_space(1))) void *global_ptr_t;
    constexpr int ROWS = kLdRows + kLoraRank;                     // staged rows: X rows first, then A rows
    constexpr int UPW = ROWS / 8 / 4;                             // copy instructions per wave and step: eight rows each
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int lrow = lane & 31, lhalf = lane >> 5;
    const int64_t m0 = (int64_t)blockIdx.x * kLdRows;
    const int step0 = blockIdx.y * steps_per_split;
    const int ksteps_all = (int)((K + 63) >> 6);                  // the last step may be partly past K (K % 16 == 0)
    const int nsteps = min(steps_per_split, ksteps_all - step0);
    // lane l of unit u copies row 8 u + l / 8, the chunk whose slot (lds_chunk_off) is l % 8
    const uint16_t *src[UPW];
    int kc[UPW];
#pragma unroll
    for (int i = 0; i < UPW; ++i) {
        const int row = 8 * (wave + 4 * i) + (lane >> 3), c = (lane & 7) ^ swz_key(row);
        src[i] = (row < kLdRows ? x + min(m0 + row, M - 1) * ldx              // rows past the end repeat the last one (never used)
                                : a + (int64_t)(row - kLdRows) * K) + 8 * c;
        kc[i] = 8 * c;
    }
    auto copy = [&](int step) {
#pragma unroll
        for (int i = 0; i < UPW; ++i) {
            const int64_t k = (int64_t)(step0 + step) * 64;
            const void *p = k + kc[i] < K ? (const void *)(src[i] + k) : (const void *)g_zeros;
            __builtin_amdgcn_global_load_lds((global_ptr_t)p, (lds_ptr_t)(lds + (step & (kLdStages - 1)) * kLdStageBytes + (wave + 4 * i) * 1024), 16, 0, 0);
        }
    };
    float16v acc[2][2];                                           // [column tile][row tile] of this wave's 64 x 64
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[c][j][r] = 0.0f;
    for (int st = 0; st < min(nsteps, kLdStages - 1); ++st) copy(st);
    for (int st = 0; st < nsteps; ++st) {
        // this wave's copies of step st have landed when at most those of the steps behind it are outstanding
        const int behind = min(nsteps - 1, st + kLdStages - 2) - st;
        if (behind >= 2) wait_vmcnt_le<2 * UPW>();
        else if (behind == 1) wait_vmcnt_le<UPW>();
        else wait_vmcnt_le<0>();
        NVFP4_COMPILER_FENCE();
        __builtin_amdgcn_s_barrier();               // step st is in LDS, and every wave has read step st - 1
        NVFP4_COMPILER_FENCE();
        if (st + kLdStages - 1 < nsteps) copy(st + kLdStages - 1);
        const uint8_t *stage = lds + (st & (kLdStages - 1)) * kLdStageBytes;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            uint4v fx[2], fa[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) fx[j] = *(const uint4v *)(stage + lds_chunk_off(64 * wm + 32 * j + lrow, 2 * kk + lhalf));
#pragma unroll
            for (int c = 0; c < 2; ++c) fa[c] = *(const uint4v *)(stage + lds_chunk_off(kLdRows + 64 * wn + 32 * c + lrow, 2 * kk + lhalf));
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[c][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8v, fa[c]),
                                                                        __builtin_bit_cast(bf16x8v, fx[j]), acc[c][j], 0, 0, 0);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");         // (this wave's reads of the stage, before the next barrier)
    }
    // lane = output row, register r = column 8 (r / 4) + 4 lhalf + r % 4 of the 32-column tile: transposed through LDS, so
    // that a wave stores four whole 256-byte runs at a time and not thirty-two of 32 bytes
    __syncthreads();
    float4v *slab = (float4v *)(lds + wave * 16384);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                slab[(32 * j + lrow) * 16 + ((8 * c + 2 * q + lhalf) ^ (lrow & 15))] =
                    float4v{acc[c][j][4 * q], acc[c][j][4 * q + 1], acc[c][j][4 * q + 2], acc[c][j][4 * q + 3]};
    NVFP4_COMPILER_FENCE();                       // (a wave reads its own slab)
    float *pp = partial + ((int64_t)blockIdx.y * m_pad + m0 + 64 * wm) * kLoraRank + 64 * wn;
#pragma unroll
    for (int p = 0; p < 16; ++p) {
        const int row = 4 * p + (lane >> 4), c4 = lane & 15;
        *(float4v *)(pp + (int64_t)row * kLoraRank + 4 * c4) = slab[row * 16 + (c4 ^ (row & 15))];
    }
#endif
}

// T = bf16(sum over the splits, in split order)
__global__ __launch_bounds__(256) void lora_down_reduce_kernel(const float *__restrict__ partial, int splits,
                                                               int64_t m_pad, int64_t M, uint16_t *__restrict__ t)
{
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;           // four consecutive columns of one row
    if (i >= M * kLoraRank) return;
    constexpr int kMost = 16;                                                    // (lora_down_plan makes no more ranges)
    float4v p[kMost];                                                           // all loads in flight together
#pragma unroll
    for (int s = 0; s < kMost; ++s)
        if (s < splits) p[s] = *(const float4v *)(partial + (int64_t)s * m_pad * kLoraRank + i);
    float4v sum = p[0];
#pragma unroll
    for (int s = 1; s < kMost; ++s)
        if (s < splits) sum += p[s];
    *(uint2v *)(t + i) = uint2v{pack_bf16x2(sum.x, sum.y), pack_bf16x2(sum.z, sum.w)};
}

bool gemm_is_tiled(int64_t M, int64_t N, int64_t K) { return tiled_ok(M, N, K); }

// "BMxBN:workgroups" per launch, separated by spaces ("generic" for shapes that only the 64x64 tile of nvfp4_gemm_split.hip takes)
int gemm_plan_text(int64_t M, int64_t N, int64_t K, char *text, size_t text_bytes)
{
    if (!tiled_ok(M, N, K)) {
        snprintf(text, text_bytes, "generic");
        return 1;
    }
    size_t used = 0;
    int launches = 0;
    bool fits = true;
    for_each_chunk(M, N, K, [&](int64_t, int64_t, int64_t, int64_t, const LaunchPlan &p) {
        for (int i = 0; i < p.n && fits; ++i) {
            const TileShape &t = kShapes[p.part[i].kind];
            const int w = snprintf(text + used, used < text_bytes ? text_bytes - used : 0, "%s%dx%d:%lld",
                                   launches ? " " : "", t.bm, t.bn, (long long)p.part[i].tiles);
            if (w < 0 || used + (size_t)w >= text_bytes) fits = false;
            else {
                used += (size_t)w;
                ++launches;
            }
        }
    });
    return fits ? launches : -1;
}

int gemm_workgroups(int64_t M, int64_t N, int64_t K)
{
    int64_t n = 0;
    for_each_chunk(M, N, K, [&](int64_t, int64_t, int64_t, int64_t, const LaunchPlan &p) {
        for (int i = 0; i < p.n; ++i) n += p.part[i].tiles;
    });
    return (int)n;
}

static hipError_t launch_kind(TileKind kind, int epi, const GemmArgs &g, int64_t tiles, hipStream_t s)
{
    switch (kind) {
    case kTile256x256: return launch_tile_256x256(epi, g, tiles, s);
    case kTile256x192: return launch_tile_256x192(epi, g, tiles, s);
    case kTile64: return launch_tile_64x64(epi, g, tiles, s);
    default: return launch_tile_128x128(epi, g, tiles, s);
    }
}

hipError_t launch_gemm(const uint8_t *codesA, const uint8_t *scalesA, const float *gsA,
                       const uint8_t *codesW, const uint8_t *scalesW, const float *gsW, int64_t M,
                       int64_t N, int64_t K, const GemmEpilogue &ep, int *n_wg, hipStream_t s,
                       const LoraBranch &lora)
{
    GemmArgs g{codesA, scalesA, codesW, scalesW, gsA, gsW, M, N, K, ep, 0, N, 0, lora.t, lora.b, lora.scale};
    const bool with_lora = lora.t != nullptr;
    if (!tiled_ok(M, N, K)) {                            // an odd shape: 64x64 tiles throughout
        if (with_lora) return hipErrorInvalidValue;      // (no LoRA phase there; callers check gemm_is_tiled)
        const int64_t tiles = ((M + 63) / 64) * ((N + 63) / 64);
        if (n_wg) *n_wg = (int)tiles;
        const int kind = ep.out_dtype != 0 ? (kEpiBF16 | (ep.act == 1 ? kEpiGelu : 0)) : kEpiF32;
        return launch_tile_64x64(kind, g, tiles, s);
    }
    // (the tiled fp32 output never carries an activation: nvfp4_gemm has none and the fused call emits bf16)
    const int out_kind = ep.q_scale ? kEpiQuant : (ep.out_dtype != 0 ? kEpiBF16 : kEpiF32);
    const int epi = out_kind | ((ep.act == 1 && out_kind != kEpiF32) ? kEpiGelu : 0);
    const int64_t kbytes = K >> 1, kblocks = K >> 4;
    const int64_t ysize = ep.out_dtype == 0 ? 4 : 2;
    int wg_total = 0;
    hipError_t err = hipSuccess;
    for_each_chunk(M, N, K, [&](int64_t cm, int64_t, int64_t cn, int64_t, const LaunchPlan &plan) {
        for (int i = 0; i < plan.n && err == hipSuccess; ++i) {
            const SubLaunch &p = plan.part[i];
            const int64_t m_lo = cm + p.m_lo, n_lo = cn + p.n_lo;     // the sub-rectangle [m_lo, ..) x [n_lo, ..) as a problem of its own
            GemmArgs a = g;
            a.codesA = codesA + m_lo * kbytes;
            a.scalesA = scalesA + m_lo * kblocks;
            a.codesW = codesW + n_lo * kbytes;
            a.scalesW = scalesW + n_lo * kblocks;
            a.M = p.m_hi - p.m_lo;
            a.N = p.n_hi - p.n_lo;
            if (ep.Y) a.ep.Y = (uint8_t *)ep.Y + (m_lo * ep.ldy + n_lo) * ysize;
            if (ep.q_codes) {
                a.ep.q_codes = ep.q_codes + m_lo * (N >> 1) + (n_lo >> 1);
                a.ep.q_scales = ep.q_scales + m_lo * (N >> 4) + (n_lo >> 4);
            }
            a.q_pitch = N;
            a.partial_base = wg_total;
            if (with_lora) {
                a.lora_t = lora.t + m_lo * kLoraRank;
                a.lora_b = lora.b + n_lo * kLoraRank;
            }
            err = launch_kind(p.kind, epi | (with_lora ? kEpiLora : 0), a, p.tiles, s);
            wg_total += (int)p.tiles;
        }
    });
    if (err != hipSuccess) return err;
    if (n_wg) *n_wg = wg_total;
    return hipSuccess;
}

// K is cut into `splits` ranges of whole 64-k steps so that about one workgroup per compute unit runs
static void lora_down_plan(int64_t M, int64_t K, int *splits, int *steps_per_split, int64_t *m_pad)
{
    const int64_t row_tiles = (M + kLdRows - 1) / kLdRows;
    const int ksteps = (int)((K + 63) >> 6);
    int want = (int)std::max<int64_t>(1, std::min<int64_t>(16, kCUs / row_tiles));
    *steps_per_split = (ksteps + want - 1) / want;
    *splits = (ksteps + *steps_per_split - 1) / *steps_per_split;
    *m_pad = row_tiles * kLdRows;
}

size_t lora_down_workspace_bytes(int64_t M, int64_t K)
{
    int splits, sps;
    int64_t m_pad;
    lora_down_plan(M, K, &splits, &sps, &m_pad);
    return (size_t)splits * (size_t)m_pad * kLoraRank * sizeof(float);
}

hipError_t launch_lora_down(const uint16_t *x, int64_t M, int64_t K, int64_t ldx, const uint16_t *a,
                            uint16_t *t, float *workspace, hipStream_t s)
{
    int splits, sps;
    int64_t m_pad;
    lora_down_plan(M, K, &splits, &sps, &m_pad);
    dim3 grid((unsigned)(m_pad / kLdRows), (unsigned)splits);
    constexpr int smem = kLdStages * kLdStageBytes;
    static uint64_t attr_set = 0;              // the dynamic LDS limit is raised once per device
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess && ((attr_set >> (dev & 63)) & 1u) == 0) {
        e = hipFuncSetAttribute((const void *)lora_down_partial_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
        if (e == hipSuccess) attr_set |= 1ull << (dev & 63);
    }
    if (e != hipSuccess) return e;
    lora_down_partial_kernel<<<grid, 256, smem, s>>>(x, M, K, ldx, a, sps, workspace, m_pad);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    lora_down_reduce_kernel<<<(unsigned)((M * kLoraRank / 4 + 255) / 256), 256, 0, s>>>(workspace, splits, m_pad, M, t);
    return hipGetLastError();
}

}  // namespace nvfp4
