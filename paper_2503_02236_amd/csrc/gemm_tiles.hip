// Second stage of the prefill VQ-gemm: Y = X * Wd^T on v_mfma_f32_16x16x32_f16 with fp32 accumulation, Wd the fp16 weight that
// launch_dequant_ordered() has left in the workspace in the order in which this kernel's wavefronts read it.
//
// Why two stages (VQ-LLM, arXiv 2503.02236, Sec. VII-B notes that dequantization hurts the compute-bound GeMM most): with a
// 2^16-entry codebook every 16-byte operand is a random gather from L2, of which MI355X does 0.4 per clock and CU.  A fused
// 256-row tile would need one gather per lane and four matrix instructions, and every further row of tiles would repeat it.
//
// What bounds it is power: on random operands the chip clocks down until a kernel of this size sustains some 1.4 PFLOP/s,
// whatever its issue slots would allow (all-zero operands: 1.9).  So what counts is the energy per product:
//   - 16 x 16 x 32 instead of 32 x 32 x 16 matrix instructions.  Per product they read and write half as much of the accumulator
//     (2048 x 8192 x 4096, this kernel with the one and the other: 101 and 111 us on random operands, 74 and 70 on zeros);
//   - the weight does not pass through LDS.  A wavefront owns 16 NF columns that no other wavefront of the workgroup has, so
//     its operands come straight from memory into registers, one contiguous KiB per load;
//   - a workgroup has BM rows of X x 64 NF columns, and every wavefront works on all BM rows, so an operand of X that has been
//     read from LDS serves NF matrix instructions.
// X goes global -> LDS directly into a ring of four stages of 64 k; 16-byte segments are swizzled with the row so that the
// operand reads (16 lanes a pass, {0-3, 12-15, 20-27} and so on) meet no bank conflict.
//
// The main loop has one barrier per 64 k, in front of the last step whose operands have already been read.  Loads are issued
// two (weight) and three (X) stages ahead.  They are buffer loads: the compiler counts them in vmcnt one by one, while it
// takes a global_load_lds for a flat access, after which every wait is for everything; and their addresses advance in a scalar.
// The matrix instructions are asm with the accumulator as in- and output: left to the compiler, accumulators change
// registers between the copies of the loop body and are moved back at its end (some 200 moves an iteration).
//
// Against the kernel before (256 x 128 tiles of 32 x 32 x 16 instructions, both operands through LDS; gemm_dense.hip), the
// second stage alone, us: 2048 x 11008 x 4096 176 -> 150, 2048 x 4096 x 4096 67 -> 57, 1024 x 4096 x 4096 40 -> 32,
// 512 x 4096 x 4096 32 -> 21.
#include <algorithm>
#include <type_traits>

#include "vq_common.h"

namespace vq {

namespace {

constexpr int kTileStages = 4;
constexpr int kTileRowB = 128;   // bytes of a row of X in a stage

struct TilesArgs {
    const half_t *X;      // [M][K]
    const half_t *W;      // ordered (vq_common.h)
    const half_t *scale;  // [N] or null
    half_t *Y;            // [M][N]
    int M, N, K;
    int tiles_m, tiles_n;
};

typedef __attribute__((address_space(3))) void lds_void_t;

__device__ __forceinline__ int tile_swz(int row) { return (row >> 1) & 7; }

// Resident wavefronts per SIMD: what registers and LDS (kTileStages * BM * 128 bytes a workgroup) allow.
constexpr int tile_waves(int BM) { return 256 / BM; }

template <int BM, int NF>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(tile_waves(BM), tile_waves(BM)))) void gemm_tiles_kernel(TilesArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)   // (the host compiler does not know the buffer builtins)
    constexpr int MF = BM / 16, BN = 64 * NF;
    constexpr int kStage = BM * kTileRowB;
    constexpr int XL = BM / 32;             // direct-to-LDS loads per wavefront and stage: 8 rows each
    constexpr int STEPS = 2;                // steps of 32 k in a stage
    constexpr int WL = STEPS * NF;          // weight loads per wavefront and stage
    constexpr int kEvery = MF / (XL / STEPS);   // row blocks between two loads of X
    static_assert(MF % (XL / STEPS) == 0 && kTileStages == 4, "");
    extern __shared__ __align__(16) unsigned char smem[];

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int ln = lane & 15, lk = lane >> 4;

    // workgroups are dealt round-robin to the 8 compute dies: each die gets a contiguous run of tiles, column by column, so that
    // its workgroups share weight columns and rows of X in its L2
    const int n_tiles = a.tiles_m * a.tiles_n, per_die = (n_tiles + 7) / 8;
    const int t = (blockIdx.x & 7) * per_die + (blockIdx.x >> 3);
    if (t >= n_tiles) return;
    const int tile_n = t / a.tiles_m, tile_m = t % a.tiles_m;
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    const int KT = a.K / 64;

    float4_t acc[MF][NF];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NF; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;

    // X: offsets from row m0; rows past the end are the last one (never stored).  (K is small enough for 32 bits: gemm_tiles_fits)
    const int rows = min(a.M - m0, BM);
    const auto xr = __builtin_amdgcn_make_buffer_rsrc((void *)(a.X + (size_t)m0 * a.K), (short)0, (unsigned)rows * (unsigned)a.K * 2u, 0x00020000);
    unsigned xoff[XL];
#pragma unroll
    for (int p = 0; p < XL; ++p) {
        const int r = wave * (BM / 4) + p * 8 + (lane >> 3);
        xoff[p] = (unsigned)min(r, rows - 1) * (unsigned)a.K * 2u + (((lane & 7) ^ tile_swz(r)) << 4);
    }
    // weight: strips of 16 columns, the last of N perhaps narrower; strips past it are the last one (never stored)
    const int strips = (a.N + 15) / 16, strip0 = min(n0 / 16 + wave * NF, strips - 1);
    const size_t first = (size_t)strip0 * 16 * a.K, all = (size_t)a.N * a.K;
    const auto wr = __builtin_amdgcn_make_buffer_rsrc((void *)(a.W + first), (short)0,
                                                      (unsigned)(all - first < (size_t)16 * NF * a.K ? all - first : (size_t)16 * NF * a.K) * 2u, 0x00020000);
    unsigned woff[NF];
    int wstep[NF];   // bytes of a fragment: 32 k of the strip's columns
#pragma unroll
    for (int j = 0; j < NF; ++j) {
        const int strip = min(strip0 + j, strips - 1), cols = min(a.N - strip * 16, 16);
        woff[j] = (unsigned)(strip - strip0) * 32u * (unsigned)a.K + (unsigned)(lk * cols + min(ln, cols - 1)) * 16u;
        wstep[j] = cols * 64;
    }
    // (past the end of K the last stage once more, for the sake of constant counts)
    auto load_x = [&](int kt, int p) {
        unsigned char *dst = smem + (size_t)(kt % kTileStages) * kStage + (size_t)wave * (BM / 4) * kTileRowB + p * 1024;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_void_t *)dst, 16, xoff[p], min(kt, KT - 1) * 128, 0, 0);
    };
    half8_t wf[2][STEPS][NF], xf[MF];
    auto load_w = [&](int kt, int slot, int s, int j) {
        wf[slot][s][j] = __builtin_bit_cast(half8_t, __builtin_amdgcn_raw_buffer_load_b128(wr, woff[j], (min(kt, KT - 1) * STEPS + s) * wstep[j], 0));
    };
    const int swz = tile_swz(ln);   // (the same in every row block)
    auto read_x = [&](int kt, int s, int i) {
        const unsigned char *xb = smem + (size_t)(kt % kTileStages) * kStage + (size_t)(i * 16 + ln) * kTileRowB;
        xf[i] = *reinterpret_cast<const half8_t *>(xb + (((s * 4 + lk) ^ swz) << 4));
    };

    // stages 0, 1, 2 of X and 0, 1 of the weight, from stage 1 on in the main loop's order
#pragma unroll
    for (int p = 0; p < XL; ++p) load_x(0, p);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
#pragma unroll
            for (int p = 0; p < XL / STEPS; ++p) load_x(1 + q, s * (XL / STEPS) + p);
#pragma unroll
            for (int j = 0; j < NF; ++j) load_w(q, q, s, j);
            __builtin_amdgcn_sched_barrier(0);
        }
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * (XL + WL)) : "memory");
#pragma unroll
    for (int i = 0; i < MF; ++i) read_x(0, 0, i);

    auto stage = [&](int kt, auto slot_tag) {
        constexpr int slot = decltype(slot_tag)::value;
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            if (s == STEPS - 1) {
                // Stage kt + 1 of X has landed: later than its last load are those of one whole stage and of the steps of this one so
                // far (and the weight loads behind it, which are not counted on).  After the barrier it has for every wavefront, and
                // all have read what they need of stage kt, whose place the loads of stage kt + 4 take from the next stage on.
                constexpr int later = (XL + WL) + (XL + WL) * (STEPS - 1) / STEPS;
                static_assert(later < 64, "vmcnt has six bits");
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(later) : "memory");
            }
            // Row block by row block: its products, then its operand of the next step into the same registers, now and then a load.
#pragma unroll
            for (int i = 0; i < MF; ++i) {
#pragma unroll
                for (int jj = 0; jj < NF; ++jj) {
                    const int j = (i & 1) ? NF - 1 - jj : jj;
                    asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(acc[i][j]) : "v"(wf[slot][s][j]), "v"(xf[i]));
                }
                read_x(s == STEPS - 1 ? kt + 1 : kt, s == STEPS - 1 ? 0 : s + 1, i);
                if (i % kEvery == 0) load_x(kt + kTileStages - 1, s * (XL / STEPS) + i / kEvery);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int j = 0; j < NF; ++j) load_w(kt + 2, slot, s, j);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    int kt = 0;
    for (; kt + 1 < KT; kt += 2) {
        stage(kt, std::integral_constant<int, 0>{});
        stage(kt + 1, std::integral_constant<int, 1>{});
    }
    if (kt < KT) stage(kt, std::integral_constant<int, 0>{});
    // The nops: the compiler does not know that the accumulators come from matrix instructions that may still be under way.  Every
    // accumulator then passes through an (empty) statement that cannot change places with this one, so that nothing reads it earlier.
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier\n\ts_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NF; ++j) asm volatile("" : "+a"(acc[i][j]));

    // An accumulator holds Y^T: lane (ln, lk), register r is row m = ln, column n = 4 lk + r of its 16 x 16 block.  Scaled and
    // rounded, blocks of kRows rows go through a private LDS region of the wavefront (rows padded by 16 bytes) and leave as 16
    // bytes per lane.
    const int wn0 = n0 + wave * NF * 16;
    float sc[NF][4];
#pragma unroll
    for (int j = 0; j < NF; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) sc[j][r] = 1.f;
    if (a.scale) {
#pragma unroll
        for (int j = 0; j < NF; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) sc[j][r] = (float)a.scale[min(wn0 + j * 16 + lk * 4 + r, a.N - 1)];
    }
    if ((a.N & 7) == 0) {
        constexpr int kOutRowB = NF * 32 + 16, kSegs = 2 * NF;
        constexpr int kRows = BM < 64 ? BM : 4 * 128 * kOutRowB <= kTileStages * kStage && BM >= 128 ? 128 : 64;
        static_assert(4 * kRows * kOutRowB <= kTileStages * kStage, "output staging must fit the ring's LDS");
        unsigned char *out = smem + (size_t)wave * kRows * kOutRowB;
#pragma unroll
        for (int c = 0; c < BM / kRows; ++c) {
#pragma unroll
            for (int i = 0; i < kRows / 16; ++i)
#pragma unroll
                for (int j = 0; j < NF; ++j) {
                    half4_t o;
#pragma unroll
                    for (int r = 0; r < 4; ++r) o[r] = (half_t)(acc[c * (kRows / 16) + i][j][r] * sc[j][r]);
                    *reinterpret_cast<half4_t *>(out + (i * 16 + ln) * kOutRowB + (j * 16 + lk * 4) * 2) = o;
                }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the same wavefront wrote what it now reads
            for (int q = lane; q < kRows * kSegs; q += 64) {
                const int row = q / kSegs, seg = q % kSegs;
                const uint4 v = *reinterpret_cast<const uint4 *>(out + row * kOutRowB + seg * 16);
                const int m = m0 + c * kRows + row, n = wn0 + seg * 8;
                if (m < a.M && n < a.N) *reinterpret_cast<uint4 *>(a.Y + (size_t)m * a.N + n) = v;
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
    } else {
        // rows of Y are not 16-byte aligned: element stores
#pragma unroll
        for (int i = 0; i < MF; ++i) {
            const int m = m0 + i * 16 + ln;
            if (m >= a.M) continue;
#pragma unroll
            for (int j = 0; j < NF; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int n = wn0 + j * 16 + lk * 4 + r;
                    if (n < a.N) a.Y[(size_t)m * a.N + n] = (half_t)(acc[i][j][r] * sc[j][r]);
                }
        }
    }
#endif
}

template <int BM, int NF>
int run_tiles(TilesArgs a, hipStream_t s) {
    constexpr int BN = 64 * NF;
    a.tiles_m = (a.M + BM - 1) / BM;
    a.tiles_n = (a.N + BN - 1) / BN;
    constexpr size_t lds = (size_t)kTileStages * BM * kTileRowB;
    static KernelSetup setup;
    if (int st = kernel_setup(reinterpret_cast<const void *>(&gemm_tiles_kernel<BM, NF>), lds, false, setup)) return st;
    const int n_tiles = a.tiles_m * a.tiles_n;
    gemm_tiles_kernel<BM, NF><<<(n_tiles + 7) / 8 * 8, 256, lds, s>>>(a);
    return launch_status();
}

}  // namespace

// Offsets inside a tile (256 rows of X or 256 columns of the weight) are 32-bit.
bool gemm_tiles_fits(int K) { return K % 64 == 0 && K <= (1 << 22); }

// Estimated time in us and the tile with the least, by measurement of all eight over 156 products (N 256 .. 11008, K 512 .. 11008,
// 257 .. 4096 tokens): a workgroup alone on its CU takes kAlone[0] per 4096 k and kAlone[1] besides; with more of the 256 CUs busy the
// chip clocks down, to 0.87 of that speed when all are; more than one workgroup a CU, where two or more fit, overlap a
// little (kOverlap).  Over 2850 other products (N 64 .. 11008, K 256 .. 11008, 257 .. 4096 tokens) the tile picked takes 1.1 % more than the best
// on average and 16 % or more in the worst hundredth: below K = 512, where the output counts, and for weights of more than 64 M elements,
// which a tile of few columns reads from memory too often (11008 x 11008, 677 tokens 167 / 224); elsewhere 0.7 % and 10 %.
double gemm_tiles_time(int M, int N, int K, int *pick) {
    static const int kTile[8][2] = {{256, 256}, {256, 192}, {128, 256}, {128, 192}, {128, 128}, {128, 64}, {64, 128}, {64, 64}};
    static const double kAlone[8][2] = {{65, 7}, {55, 6}, {37, 3.2}, {30, 3.2}, {22.5, 1.6}, {17.5, 1.8}, {15.5, 1.8}, {11.8, 1.6}};
    static const double kOverlap[8] = {1, 1, 0.92, 0.92, 0.92, 0.95, 0.79, 0.95};
    const auto slower = [](double busy) { return std::max(1.0, 0.54 + 0.6 * busy); };
    double best = 1e300;
    for (int t = 0; t < 8; ++t) {
        const long tiles = (((long)M + kTile[t][0] - 1) / kTile[t][0]) * (((long)N + kTile[t][1] - 1) / kTile[t][1]);
        const double one = kAlone[t][0] * K / 4096 + kAlone[t][1], rest = (tiles % 256) / 256.0;
        double time = one * ((tiles / 256) * slower(1) + (rest > 0 ? slower(rest) : 0));
        if (tiles > 256) time *= kOverlap[t];
        if (time < best) {
            best = time;
            if (pick) *pick = t;
        }
    }
    return best;
}

int launch_gemm_tiles(const half_t *X, const half_t *W, const half_t *scale, half_t *Y, int M, int N, int K, int pick, hipStream_t s) {
    const TilesArgs a = {X, W, scale, Y, M, N, K, 0, 0};
    switch (pick) {
        case 0: return run_tiles<256, 4>(a, s);
        case 1: return run_tiles<256, 3>(a, s);
        case 2: return run_tiles<128, 4>(a, s);
        case 3: return run_tiles<128, 3>(a, s);
        case 4: return run_tiles<128, 2>(a, s);
        case 5: return run_tiles<128, 1>(a, s);
        case 6: return run_tiles<64, 2>(a, s);
        default: return run_tiles<64, 1>(a, s);
    }
}

}  // namespace vq
