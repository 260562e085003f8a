// Test-hook kernels: the dequantized operand itself (VQ-LLM Sec. II-A, dequantization:
// look up one entry per residual codebook, add them element-wise, concatenate sub-vectors),
// plus two streaming probes used to calibrate bandwidth measurements.
#include <type_traits>

#include "vq_common.h"

namespace vq {

// One thread per sub-vector: W[n][j*V .. j*V+V) = sum_r C_r[code[n][j][r]] (fp32, r ascending).
template <typename CodeT, int V, bool OUT32>
__global__ __launch_bounds__(256) void dequant_kernel(const void *__restrict__ codes,
                                                      const half_t *__restrict__ cb_all, void *__restrict__ out,
                                                      long n_vec, int R, int E, int J, int tile_n, int tile_j,
                                                      int tiles_k) {
    long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    long stride = (long)gridDim.x * blockDim.x;
    for (; i < n_vec; i += stride) {
        float acc[V];
        half_t first[V];
        // per-tile codebooks (Sec. III-B, Tbl. III): the set of the tile that holds sub-vector (n, j)
        const half_t *cb = cb_all;
        if (tile_n > 0) cb += ((size_t)((i / J) / tile_n) * tiles_k + (size_t)((i % J) / tile_j)) * ((size_t)R * E * V);
        for (int r = 0; r < R; ++r) {
            unsigned c = read_code<CodeT>(codes, (size_t)i * R + r);
            const half_t *e = cb + ((size_t)r * E + c) * V;
#pragma unroll
            for (int k = 0; k < V; ++k) {
                half_t h = e[k];
                if (r == 0) {
                    first[k] = h;
                    acc[k] = (float)h;
                } else {
                    acc[k] += (float)h;
                }
            }
        }
        if (OUT32) {
            float *o = reinterpret_cast<float *>(out) + i * V;
#pragma unroll
            for (int k = 0; k < V; ++k) o[k] = acc[k];
        } else {
            half_t *o = reinterpret_cast<half_t *>(out) + i * V;
#pragma unroll
            for (int k = 0; k < V; ++k) o[k] = (R == 1) ? first[k] : (half_t)acc[k];  // RNE
        }
    }
}

// The fp16 tile of one or two per-tensor codebooks in row order (vq_dequant, and the product of a K beyond 2^22): kDequantUnroll sub-vectors per
// thread, 256 apart, so that every load and store is coalesced.  What bounds it is one gather per code from L1 or L2, and
// for that many gathers have to be in flight: with one sub-vector per thread a thread waits for its code (a trip to memory),
// then for its entry, and is gone.  N = 11008, K = 4096: two 256-entry codebooks 27.0 -> 19.1 us, 12-bit codes 44.0 -> 38.8,
// 2^16 entries 30.3 -> 30.1 (gathers from L2 alone 24).  Non-temporal
// stores are 2 us faster here, but a product behind it then finds less of the tile in L2 and loses more than that.  Below 512
// workgroups the plain kernel has more wavefronts: N = 300, K = 1024 2.4 us, here 3.3.
constexpr int kDequantUnroll = 8;
template <typename CodeT, int V, int R>
__global__ __launch_bounds__(256) void dequant_half_kernel(const void *__restrict__ codes, const half_t *__restrict__ cb,
                                                           half_t *__restrict__ out, long n_vec, int E) {
    typedef unsigned raw_t __attribute__((ext_vector_type(V / 2)));
    static_assert(kDequantUnroll == 8, "the statements below name all of them");
    const long base = (long)blockIdx.x * (256 * kDequantUnroll) + threadIdx.x;
    auto look_up = [&](int r, unsigned c) { return *reinterpret_cast<const raw_t *>(cb + ((unsigned)(r * E) + c) * (unsigned)V); };
    auto add = [](raw_t x, raw_t y) {   // RNE of the fp32 sum
        typedef half_t half_v __attribute__((ext_vector_type(V)));
        half_v a = __builtin_bit_cast(half_v, x);
        const half_v b = __builtin_bit_cast(half_v, y);
#pragma unroll
        for (int k = 0; k < V; ++k) a[k] = (half_t)((float)a[k] + (float)b[k]);
        return __builtin_bit_cast(raw_t, a);
    };
    raw_t *o = reinterpret_cast<raw_t *>(out);
    if ((long)(blockIdx.x + 1) * (256 * kDequantUnroll) > n_vec) {   // the last workgroup
        for (long i = base; i < n_vec; i += 256) {
            raw_t e = look_up(0, read_code<CodeT>(codes, (size_t)i * R));
            if (R == 2) e = add(e, look_up(R - 1, read_code<CodeT>(codes, (size_t)i * R + R - 1)));
            o[i] = e;
        }
        return;
    }
    unsigned c[kDequantUnroll][R];
#pragma unroll
    for (int u = 0; u < kDequantUnroll; ++u)
#pragma unroll
        for (int r = 0; r < R; ++r) c[u][r] = read_code<CodeT>(codes, (size_t)(base + u * 256) * R + r);
    // the empty statements keep the compiler from taking one sub-vector after the other to save registers
    raw_t e[R][kDequantUnroll];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        asm volatile("" : "+v"(c[0][r]), "+v"(c[1][r]), "+v"(c[2][r]), "+v"(c[3][r]), "+v"(c[4][r]), "+v"(c[5][r]), "+v"(c[6][r]), "+v"(c[7][r]));
#pragma unroll
        for (int u = 0; u < kDequantUnroll; ++u) e[r][u] = look_up(r, c[u][r]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        asm volatile("" : "+v"(e[r][0]), "+v"(e[r][1]), "+v"(e[r][2]), "+v"(e[r][3]), "+v"(e[r][4]), "+v"(e[r][5]), "+v"(e[r][6]), "+v"(e[r][7]));
#pragma unroll
    for (int u = 0; u < kDequantUnroll; ++u) o[base + u * 256] = R == 2 ? add(e[0][u], e[R - 1][u]) : e[0][u];
}

template <typename CodeT, int V>
static void run_dequant_half(const vq_weight_t *w, half_t *W, long n_vec, hipStream_t s) {
    const long blocks = (n_vec + 256 * kDequantUnroll - 1) / (256 * kDequantUnroll);
    if (w->n_codebooks == 1) {
        if constexpr (!std::is_same<CodeT, Code12>::value || V == 4)   // (dequant_in_eights)
            dequant_half_kernel<CodeT, V, 1><<<(int)blocks, 256, 0, s>>>(w->codes, (const half_t *)w->codebooks, W, n_vec, w->n_entries);
    } else {
        dequant_half_kernel<CodeT, V, 2><<<(int)blocks, 256, 0, s>>>(w->codes, (const half_t *)w->codebooks, W, n_vec, w->n_entries);
    }
}

// Where the kernel above runs.  Not for one 12-bit codebook of 8-vectors, the one format that it slows down (N = K = 4096, plain
// kernel / eights: 11.9 / 14.1 us, N = 11008 27.3 / 28.3; two codebooks 18.0 / 16.9, 4-vectors 16.2 / 15.2; why was not established).
bool dequant_in_eights(const vq_weight_t *w) {
    const long n_vec = (long)w->N * (w->K / w->v);
    return w->cb_tile_n == 0 && w->n_codebooks <= 2 && !(w->code_bits == 12 && w->v == 8 && w->n_codebooks == 1) &&
           n_vec >= 512L * 256 * kDequantUnroll && n_vec < (1L << 40);
}

int launch_dequant(const vq_weight_t *w, void *W, int out_fp32, hipStream_t s) {
    long n_vec = (long)w->N * (w->K / w->v);
    if (!out_fp32 && dequant_in_eights(w)) {
        half_t *o = (half_t *)W;
        if (w->code_bits == 8) w->v == 8 ? run_dequant_half<uint8_t, 8>(w, o, n_vec, s) : run_dequant_half<uint8_t, 4>(w, o, n_vec, s);
        else if (w->code_bits == 12) w->v == 8 ? run_dequant_half<Code12, 8>(w, o, n_vec, s) : run_dequant_half<Code12, 4>(w, o, n_vec, s);
        else w->v == 8 ? run_dequant_half<uint16_t, 8>(w, o, n_vec, s) : run_dequant_half<uint16_t, 4>(w, o, n_vec, s);
        return launch_status();
    }
    int blocks = (int)((n_vec + 255) / 256 < 65536 ? (n_vec + 255) / 256 : 65536);
    const int J = w->K / w->v, tile_n = w->cb_tile_n, tile_j = tile_n > 0 ? w->cb_tile_k / w->v : 1,
              tiles_k = tile_n > 0 ? w->K / w->cb_tile_k : 1;
#define VQ_DQ(CT, V)                                                                                            \
    do {                                                                                                        \
        if (out_fp32)                                                                                           \
            dequant_kernel<CT, V, true><<<blocks, 256, 0, s>>>(w->codes, (const half_t *)w->codebooks, W, \
                                                               n_vec, w->n_codebooks, w->n_entries, J, tile_n, tile_j, tiles_k); \
        else                                                                                                    \
            dequant_kernel<CT, V, false><<<blocks, 256, 0, s>>>(w->codes, (const half_t *)w->codebooks, W, \
                                                                n_vec, w->n_codebooks, w->n_entries, J, tile_n, tile_j, tiles_k); \
    } while (0)
    if (w->code_bits == 8) {
        if (w->v == 8) VQ_DQ(uint8_t, 8); else VQ_DQ(uint8_t, 4);
    } else if (w->code_bits == 12) {
        if (w->v == 8) VQ_DQ(Code12, 8); else VQ_DQ(Code12, 4);
    } else {
        if (w->v == 8) VQ_DQ(uint16_t, 8); else VQ_DQ(uint16_t, 4);
    }
#undef VQ_DQ
    return launch_status();
}

// The fp16 weight in operand order (vq_common.h), the first stage of the prefill product; the same bits as above.
struct OrderedArgs {
    const void *codes;
    const half_t *cb;
    half_t *out;
    int N, K, E;
    int tile_n, tile_k, tiles_k;   // per-tile codebooks (tile_n 0: per tensor)
};

// UNITS groups of 8 k per thread.  A wavefront takes 16 rows (a strip); with 8 units a lane has 64 k of a row, four lanes a row's
// 256, and reads its codes as whole words; every store of the wavefront is four runs of 256 bytes.  Eight lookups are in flight per
// thread and codebook: what bounds it is one gather per code from L1 or L2, or the stores.  2 units: the same with a thread per 16
// k and code by code, for small weights, which have too few wavefronts otherwise.
template <typename CodeT, int V, int R, int UNITS>
__global__ __launch_bounds__(256) void dequant_ordered_kernel(OrderedArgs a) {
    constexpr int BITS = std::is_same<CodeT, Code12>::value ? 12 : 8 * (int)sizeof(typename std::conditional<std::is_same<CodeT, Code12>::value, char, CodeT>::type);
    constexpr int H = 8 / V;                 // sub-vectors per unit
    constexpr int WORDS = 64 / V * R * BITS / 32;   // code words of 64 k
    const int lane = threadIdx.x & 63, ln = lane & 15, part = lane >> 4;
    const int KC = a.K / 64, groups = UNITS == 8 ? (KC + 3) / 4 : KC;   // wavefronts per strip
    const int id = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int strip = id / groups, chunk = UNITS == 8 ? (id - strip * groups) * 4 + part : id - strip * groups;
    const int row = strip * 16 + ln, cols = min(a.N - strip * 16, 16);
    if (row >= a.N || chunk >= KC) return;
    const int u0 = UNITS == 8 ? 0 : part * UNITS;   // first unit of this thread in its 64 k
    const size_t first = (size_t)row * (a.K / V) + (size_t)chunk * (64 / V);   // sub-vector (of 64 k)

    unsigned code[UNITS * H * R];
    if constexpr (UNITS == 8) {
        uint32_t w[WORDS + 1];
        const uint32_t *src = reinterpret_cast<const uint32_t *>(reinterpret_cast<const unsigned char *>(a.codes) + first * R * BITS / 8);
#pragma unroll
        for (int i = 0; i < WORDS; ++i) w[i] = src[i];
        w[WORDS] = 0;
#pragma unroll
        for (int i = 0; i < UNITS * H * R; ++i) {
            const int b = i * BITS;
            uint32_t c = w[b / 32] >> (b % 32);
            if (b % 32 + BITS > 32) c = __builtin_amdgcn_alignbit(w[b / 32 + 1], w[b / 32], b % 32);
            code[i] = c & ((1u << BITS) - 1u);
        }
    } else {
#pragma unroll
        for (int i = 0; i < UNITS * H * R; ++i) code[i] = read_code<CodeT>(a.codes, (first + u0 * H) * R + i);
    }

    typedef unsigned raw_t __attribute__((ext_vector_type(V / 2)));
    const half_t *cb = a.cb;   // (a tile of codebooks is a multiple of 16 rows x 64 k: check_weight)
    if (a.tile_n > 0) cb += ((size_t)(strip * 16 / a.tile_n) * a.tiles_k + (size_t)(chunk * 64 / a.tile_k)) * ((size_t)R * a.E * V);
    auto look_up = [&](int i, int r) {   // i: sub-vector of this thread
        return *reinterpret_cast<const raw_t *>(cb + ((unsigned)(r * a.E) + code[i * R + r]) * (unsigned)V);
    };
    constexpr int AT = R <= 2 ? UNITS : 2;   // units looked up together
    half_t *out = a.out + (size_t)strip * 16 * a.K + (size_t)chunk * 64 * cols + ln * 8;
#pragma unroll
    for (int g = 0; g < UNITS; g += AT) {
        raw_t e[R][AT * H];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int i = 0; i < AT * H; ++i) e[r][i] = look_up(g * H + i, r);
        if constexpr (UNITS == 8) __builtin_amdgcn_sched_barrier(0);   // (or one lookup after the other, to save registers)
#pragma unroll
        for (int u = 0; u < AT; ++u) {
            V16 o;
#pragma unroll
            for (int h = 0; h < H; ++h) {
                typedef half_t half_v __attribute__((ext_vector_type(V)));
                half_v sum = __builtin_bit_cast(half_v, e[0][u * H + h]);
                if constexpr (R > 1) {   // RNE of the fp32 sum, r ascending
                    float f[V];
#pragma unroll
                    for (int k = 0; k < V; ++k) f[k] = (float)sum[k];
#pragma unroll
                    for (int r = 1; r < R; ++r) {
                        const half_v x = __builtin_bit_cast(half_v, e[r][u * H + h]);
#pragma unroll
                        for (int k = 0; k < V; ++k) f[k] += (float)x[k];
                    }
#pragma unroll
                    for (int k = 0; k < V; ++k) sum[k] = (half_t)f[k];
                }
                const raw_t raw = __builtin_bit_cast(raw_t, sum);
#pragma unroll
                for (int k = 0; k < V / 2; ++k) o.w[h * (V / 2) + k] = raw[k];
            }
            *reinterpret_cast<uint4 *>(out + (size_t)(u0 + g + u) * 8 * cols) = o.u;
        }
    }
}

template <typename CodeT, int V, int R>
static int run_dequant_ordered(const OrderedArgs &a, hipStream_t s) {
    const long strips = (a.N + 15) / 16, KC = a.K / 64, waves8 = strips * ((KC + 3) / 4);
    // below 2048 wavefronts of eight units a quarter of the work per thread
    if (waves8 >= 2048)
        dequant_ordered_kernel<CodeT, V, R, 8><<<(unsigned)((waves8 + 3) / 4), 256, 0, s>>>(a);
    else
        dequant_ordered_kernel<CodeT, V, R, 2><<<(unsigned)((strips * KC + 3) / 4), 256, 0, s>>>(a);
    return launch_status();
}

template <typename CodeT, int V>
static int run_dequant_ordered(const vq_weight_t *w, const OrderedArgs &a, hipStream_t s) {
    switch (w->n_codebooks) {
        case 1: return run_dequant_ordered<CodeT, V, 1>(a, s);
        case 2: return run_dequant_ordered<CodeT, V, 2>(a, s);
        case 3: return run_dequant_ordered<CodeT, V, 3>(a, s);
        default: return run_dequant_ordered<CodeT, V, 4>(a, s);
    }
}

int launch_dequant_ordered(const vq_weight_t *w, half_t *W, hipStream_t s) {
    const OrderedArgs a = {w->codes, (const half_t *)w->codebooks, W, w->N, w->K, w->n_entries,
                           w->cb_tile_n, w->cb_tile_n > 0 ? w->cb_tile_k : 1, w->cb_tile_n > 0 ? w->K / w->cb_tile_k : 1};
    if (w->code_bits == 8) return w->v == 8 ? run_dequant_ordered<uint8_t, 8>(w, a, s) : run_dequant_ordered<uint8_t, 4>(w, a, s);
    if (w->code_bits == 12) return w->v == 8 ? run_dequant_ordered<Code12, 8>(w, a, s) : run_dequant_ordered<Code12, 4>(w, a, s);
    return w->v == 8 ? run_dequant_ordered<uint16_t, 8>(w, a, s) : run_dequant_ordered<uint16_t, 4>(w, a, s);
}

// One thread per (b, h, t, p): copies entry k/v_codebooks[h][g(p)][code] verbatim.
__global__ __launch_bounds__(256) void kv_dequant_kernel(const uint8_t *__restrict__ codes,
                                                         const uint16_t *__restrict__ cb,
                                                         uint16_t *__restrict__ out, long n_vec, int H, int T,
                                                         int P, int v, int E, int G) {
    long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    long stride = (long)gridDim.x * blockDim.x;
    for (; i < n_vec; i += stride) {
        int p = (int)(i % P);
        long bht = i / P;
        int h = (int)((bht / T) % H);
        int g = (int)(((long)p * G) / P);
        const uint16_t *e = cb + (((size_t)h * G + g) * E + codes[i]) * v;
        for (int k = 0; k < v; ++k) out[i * v + k] = e[k];
    }
}

int launch_kv_dequant(const vq_kv_t *kv, int which, void *out, hipStream_t s) {
    int P = kv->D / kv->v;
    long n_vec = (long)kv->B * kv->H * kv->T * P;
    int blocks = (int)((n_vec + 255) / 256 < 65536 ? (n_vec + 255) / 256 : 65536);
    kv_dequant_kernel<<<blocks, 256, 0, s>>>((const uint8_t *)(which ? kv->v_codes : kv->k_codes),
                                             (const uint16_t *)(which ? kv->v_codebooks : kv->k_codebooks),
                                             (uint16_t *)out, n_vec, kv->H, kv->T, P, kv->v, kv->n_entries,
                                             kv->cb_groups);
    return launch_status();
}

// ---- measurement probes: 128-bit streaming copy / read-reduce -------------------------------

__global__ __launch_bounds__(256) void probe_copy_kernel(uint4 *__restrict__ dst, const uint4 *__restrict__ src,
                                                         size_t n16) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n16; i += stride) dst[i] = src[i];
}

// A contiguous chunk per workgroup, eight independent non-temporal 16-byte loads in flight per thread: the
// fastest plain read of a large buffer found on this chip (grid-stride order and ordinary loads are 10 - 15 %
// slower).
__global__ __launch_bounds__(256) void probe_read_kernel(const uint4 *__restrict__ src, size_t n16,
                                                         uint4 *__restrict__ sink) {
    typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
    constexpr int U = 8;
    const size_t per_wg = (n16 + gridDim.x - 1) / gridDim.x;
    const size_t begin = (size_t)blockIdx.x * per_wg, end = begin + per_wg < n16 ? begin + per_wg : n16;
    const u32x4_t *p = reinterpret_cast<const u32x4_t *>(src);
    u32x4_t a = {0, 0, 0, 0};
    size_t i = begin + threadIdx.x;
    for (; i + (U - 1) * 256 < end; i += U * 256) {
        u32x4_t v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = __builtin_nontemporal_load(p + i + u * 256);
#pragma unroll
        for (int u = 0; u < U; ++u) a ^= v[u];
    }
    for (; i < end; i += 256) a ^= __builtin_nontemporal_load(p + i);
    // fold the block into one value so the loads cannot be removed
    __shared__ uint4 red[256];
    red[threadIdx.x] = make_uint4(a.x, a.y, a.z, a.w);
    __syncthreads();
    if (threadIdx.x == 0) {
        uint4 t = make_uint4(0, 0, 0, 0);
        for (int k = 0; k < 256; ++k) { t.x ^= red[k].x; t.y ^= red[k].y; t.z ^= red[k].z; t.w ^= red[k].w; }
        sink[blockIdx.x] = t;
    }
}

// Register-resident matrix-core loop: 8 independent 32x32x16 fp16 MFMA accumulator chains per wavefront,
// no memory traffic.  What the fp16 matrix cores sustain on this chip, for the second roofline fraction.
// RANDOM: four operand pairs of pseudo-random halves in [-1, 1) per lane, taken in turn, as in a gemm on
// real data; the smooth operands of the other form (one pair, values that barely differ between lanes)
// toggle far fewer bits, and the chip clocks higher on them.
template <bool RANDOM>
__global__ __launch_bounds__(256) void probe_mfma_kernel(int iters, float *sink) {
    float16_t acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
    constexpr int P = RANDOM ? 4 : 1;
    half8_t a[P], b[P];
    uint32_t h = (blockIdx.x * 256u + threadIdx.x) * 2654435761u + 12345u;
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (RANDOM) {
                h = h * 1664525u + 1013904223u;
                a[p][i] = (half_t)(((int)(h >> 16) - 32768) * (1.f / 32768.f));
                h = h * 1664525u + 1013904223u;
                b[p][i] = (half_t)(((int)(h >> 16) - 32768) * (1.f / 32768.f));
            } else {
                a[p][i] = (half_t)(threadIdx.x * 0.001f);
                b[p][i] = (half_t)(i * 0.01f);
            }
        }
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[i % P], b[(i / 2) % P], acc[i], 0, 0, 0);
    }
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) t += acc[i][0];
    if (t == 12345.f) sink[0] = t;  // keeps the loop alive; practically never stores
}

// The same eight MFMAs per iteration, but fed the way a gemm feeds them: six fresh operands (four of one
// matrix, two of the other) read from LDS for every iteration, random halves in [-1, 1).  32 KiB of LDS per
// workgroup, so four workgroups (16 wavefronts) share a CU and cover each other's LDS latency.  No global
// memory traffic.  This is what the matrix cores sustain on operands that change with every instruction.
__global__ __launch_bounds__(256) void probe_mfma_lds_kernel(int iters, float *sink) {
    __shared__ __align__(16) half_t pool[16384];
    uint32_t h = (blockIdx.x * 256u + threadIdx.x) * 2654435761u + 977u;
    for (int i = threadIdx.x; i < 16384; i += 256) {
        h = h * 1664525u + 1013904223u;
        pool[i] = (half_t)(((int)(h >> 16) - 32768) * (1.f / 32768.f));
    }
    __syncthreads();
    float16_t acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
    const unsigned char *base = reinterpret_cast<const unsigned char *>(pool) + (threadIdx.x & 63) * 16;
    unsigned off = (threadIdx.x >> 6) * 6144u;
    for (int it = 0; it < iters; ++it) {
        half8_t op[6];
#pragma unroll
        for (int q = 0; q < 6; ++q)  // a wave-wide read of 1 KiB of consecutive bytes: no bank conflicts
            op[q] = *reinterpret_cast<const half8_t *>(base + ((off + q * 1024u) & 0x7C00u));
        off += 6144u;
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(op[4 + (i & 1)], op[i >> 1], acc[i], 0, 0, 0);
    }
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) t += acc[i][0];
    if (t == 12345.f) sink[0] = t;  // keeps the loop alive; practically never stores
}

int launch_probe_mfma(int workgroups, int iters, int random_operands, void *sink, hipStream_t s) {
    if (random_operands == 2)
        probe_mfma_lds_kernel<<<workgroups, 256, 0, s>>>(iters, (float *)sink);
    else if (random_operands)
        probe_mfma_kernel<true><<<workgroups, 256, 0, s>>>(iters, (float *)sink);
    else
        probe_mfma_kernel<false><<<workgroups, 256, 0, s>>>(iters, (float *)sink);
    return launch_status();
}

int launch_probe_copy(void *dst, const void *src, size_t bytes, hipStream_t s) {
    size_t n16 = bytes / 16;
    int blocks = (int)((n16 + 255) / 256 < 4096 ? (n16 + 255) / 256 : 4096);
    probe_copy_kernel<<<blocks, 256, 0, s>>>((uint4 *)dst, (const uint4 *)src, n16);
    return launch_status();
}

int launch_probe_read(const void *src, size_t bytes, void *sink, hipStream_t s) {
    size_t n16 = bytes / 16;
    int blocks = (int)((n16 + 2047) / 2048 < 512 ? (n16 + 2047) / 2048 : 512);   // (the sink holds one value per block)
    if (blocks < 1) blocks = 1;
    probe_read_kernel<<<blocks, 256, 0, s>>>((const uint4 *)src, n16, (uint4 *)sink);
    return launch_status();
}

}  // namespace vq
