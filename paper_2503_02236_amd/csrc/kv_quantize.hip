// On-the-fly KV quantization for gfx950: the codes of new tokens' K and V vectors.
// VQ-LLM (arXiv 2503.02236) Sec. II-A (assignment step: a sub-vector is replaced by the index of its
// closest codebook entry) and Sec. VII "Quantization Overhead" (it runs for the new token in every decode
// step and for all prompt tokens in prefill).
//
// A floating-point comparison decides an integer, so order and precision are part of the definition
// (the paper gives none; this is the reading the CPU reference follows too): squared Euclidean distance
// in fp32, elements in ascending order, every subtraction, multiplication and addition rounded on its own
// (no fused multiply-add); strict "<" while walking the entries in ascending order, so ties go to the smallest index.
//
// Three kernels with the same codes: kv_quantize_scan_kernel computes every distance, a wavefront per sub-vector (decode
// steps), kv_quantize_lane_kernel does so with a lane per sub-vector or a few (small codebooks), and kv_quantize_mfma_kernel lets the
// matrix cores rule out all but eight entries (prompts).
#include <algorithm>

#include "vq_common.h"

namespace vq {

struct KvQuantArgs {
    const half_t *x[2];    // K, V: [B][H][n_new][D]
    const half_t *cb[2];   // [H][G][E][v]
    uint8_t *codes[2];     // [B][H][T][D/v]
    int H, T, D, P, E, G, n_new, pos;
    int tokens;            // new tokens per workgroup
    int PG;                // sub-vectors per group of the codebook
    unsigned pg_inverse;   // kvq_inverse(PG) (matrix-core kernel)
    int log_lanes;         // lanes that share an item (kv_quantize_lane_kernel)
    int share;             // workgroups that share a token range (kv_quantize_scan_kernel)
};

// A sub-vector (V halves, aligned) in the low halves of 16 bytes, the rest zero.
template <int V>
__device__ __forceinline__ V16 kvq_load(const void *p) {
    V16 r;
    if constexpr (V == 8) {
        r = ld16(p);
    } else if constexpr (V == 4) {
        const V8 t = ld8(p);
        r.u = make_uint4(t.w[0], t.w[1], 0, 0);
    } else {
        r.u = make_uint4(*reinterpret_cast<const uint32_t *>(p), 0, 0, 0);
    }
    return r;
}

// x - c of two pairs of halves in fp32: a fused c * (-1) + x, whose product is exact, so that it rounds once like the
// subtraction; it takes the halves as they are.
__device__ __forceinline__ float mix_diff_lo(uint32_t x, uint32_t c) {
    float r;
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,1]" : "=v"(r) : "v"(c), "v"(x));
    return r;
}
__device__ __forceinline__ float mix_diff_hi(uint32_t x, uint32_t c) {
    float r;
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,1] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(c), "v"(x));
    return r;
}

// The definition's distance of x and c (V halves each).
template <int V>
__device__ __forceinline__ float kvq_exact(const V16 &x, const V16 &c) {
#pragma clang fp contract(off)
    float d = 0.f;
#pragma unroll
    for (int i = 0; i < V / 2; ++i) {
        const float lo = mix_diff_lo(x.w[i], c.w[i]), hi = mix_diff_hi(x.w[i], c.w[i]);
        const float s0 = lo * lo, s1 = hi * hi;
        d = i == 0 ? s0 : d + s0;
        d = d + s1;
    }
    return d;
}

// Smallest value over the wavefront, and the smallest index e among the lanes that hold it (64 lanes active, e < 256
// with e % 64 == lane): the minimum by lane permutes on the vector ALU, the index from the mask of its holders.
template <int CTRL>
__device__ __forceinline__ float dpp_min_step(float x) {
    const int y = __builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(x), CTRL, 0xF, 0xF, false);
    return fminf(x, __int_as_float(y));
}
__device__ __forceinline__ int kvq_wave_argmin(float d, int e) {
    float m = dpp_min_step<0xB1>(d);    // quad_perm [1,0,3,2]
    m = dpp_min_step<0x4E>(m);          // quad_perm [2,3,0,1]
    m = dpp_min_step<0x141>(m);         // row_half_mirror
    m = dpp_min_step<0x140>(m);         // row_mirror: rows of 16 done
    const int mi = __float_as_int(m);
    const float m0 = fminf(__int_as_float(__builtin_amdgcn_readlane(mi, 0)), __int_as_float(__builtin_amdgcn_readlane(mi, 16)));
    const float m1 = fminf(__int_as_float(__builtin_amdgcn_readlane(mi, 32)), __int_as_float(__builtin_amdgcn_readlane(mi, 48)));
    m = fminf(m0, m1);
    unsigned long long at = __ballot(d == m);
    int r = __builtin_amdgcn_readlane(e, __ffsll((long long)at) - 1);
    for (at &= at - 1; at; at &= at - 1) r = min(r, __builtin_amdgcn_readlane(e, __ffsll((long long)at) - 1));
    return r;
}

// Decode steps (few new tokens).  A wavefront takes the sub-vectors of one group: every lane holds four entries of the
// group's codebook in registers (entry lane + 64 k, straight from memory: nothing is staged, so a codebook that serves a
// single sub-vector -- coupled quantization -- is read once and used once) and the sub-vectors come one after the other.
// Bound: the latency of two dependent loads and, per sub-vector, four distances and one reduction over the lanes.  One
// token of B3 H32 with 32 codebooks per head and side: 4.4 us (5.3 with a workgroup per
// token range), where staging both sides' codebooks in LDS took 14.7.  SHARED: several workgroups share a token range.
template <int V, bool SHARED>
__global__ __launch_bounds__(512) void kv_quantize_scan_kernel(KvQuantArgs a) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    constexpr int NW = 8;
    const int bh = blockIdx.x, h = bh % a.H, side = SHARED ? blockIdx.z & 1 : blockIdx.z;
    const int t0 = blockIdx.y * a.tokens, nt = min(a.tokens, a.n_new - t0);
    const half_t *src = a.cb[side] + (size_t)h * a.G * a.E * V;
    const half_t *xs = a.x[side] + ((size_t)bh * a.n_new + t0) * a.D;
    uint8_t *dst = a.codes[side] + ((size_t)bh * a.T + a.pos + t0) * a.P;
    const int n_items = nt * a.PG;                // per group
    const int all = SHARED ? NW * a.share : NW;   // wavefronts of the workgroups that share these tokens
    const int R = max(1, all / a.G);              // wavefronts that share a group
    for (int u = (SHARED ? NW * (blockIdx.z >> 1) : 0) + wave; u < a.G * R; u += all) {
        const int g = u / R;
        V16 c[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) c[k] = kvq_load<V>(src + ((size_t)g * a.E + min(lane + 64 * k, a.E - 1)) * V);
        for (int i = u % R; i < n_items; i += R) {
            const int t = i / a.PG, p = g * a.PG + (i - t * a.PG);
            const V16 x = kvq_load<V>(xs + (size_t)t * a.D + p * V);   // the same for all lanes
            float bd = INFINITY;
            int be = lane;                        // (nothing is closer than infinity: entry 0, as lane 0 has it)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float d = kvq_exact<V>(x, c[k]);
                const bool closer = d < bd && lane + 64 * k < a.E;
                be = closer ? lane + 64 * k : be;
                bd = closer ? d : bd;
            }
            const int code = kvq_wave_argmin(bd, be);
            if (lane == 0) dst[(size_t)t * a.P + p] = (uint8_t)code;
        }
    }
}

// Small codebooks, and medium ones with few items.  A lane takes an item and walks over the entries in LDS, TOK items (of the
// same position in different tokens) at a time; where a workgroup has few items, 2^log_lanes lanes share one, each taking every
// 2^log_lanes-th entry.  Groups lie an entry more than their length apart, so that lanes of different groups read different
// banks.  Bound: vector issue, about 4 + 2.5 V instructions per (item, entry); the matrix-core kernel spends 100 or more on
// an item whatever E is.
template <int V, int TOK>
__global__ __launch_bounds__(256) void kv_quantize_lane_kernel(KvQuantArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    half_t *cb = reinterpret_cast<half_t *>(smem);   // [G][E + 1][V]
    const int tid = threadIdx.x;
    const int bh = blockIdx.x, h = bh % a.H, side = blockIdx.z;
    const int t0 = blockIdx.y * a.tokens, nt = min(a.tokens, a.n_new - t0);
    const half_t *src = a.cb[side] + (size_t)h * a.G * a.E * V;
    const half_t *xs = a.x[side] + ((size_t)bh * a.n_new + t0) * a.D;
    uint8_t *dst = a.codes[side] + ((size_t)bh * a.T + a.pos + t0) * a.P;
    for (int i = tid; i < a.G * a.E; i += 256) {
        const V16 c = kvq_load<V>(src + (size_t)i * V);
#pragma unroll
        for (int k = 0; k < V / 2; ++k) reinterpret_cast<uint32_t *>(cb + (size_t)(i + i / a.E) * V)[k] = c.w[k];
    }
    __syncthreads();
    if constexpr (TOK > 1) {
        const int rows = 256 / a.P, row = tid / a.P, p = tid - row * a.P;   // tokens side by side; this lane's position
        if (row >= rows) return;
        const half_t *grp = cb + (size_t)(p / a.PG) * (a.E + 1) * V;
        for (int t = row; t < nt; t += rows * TOK) {
            V16 x[TOK];
            float bd[TOK];
            int be[TOK];
#pragma unroll
            for (int k = 0; k < TOK; ++k) {
                x[k] = kvq_load<V>(xs + (size_t)min(t + k * rows, nt - 1) * a.D + p * V);
                bd[k] = INFINITY;
                be[k] = 0;
            }
            for (int e = 0; e < a.E; ++e) {
                const V16 c = kvq_load<V>(grp + (size_t)e * V);
#pragma unroll
                for (int k = 0; k < TOK; ++k) {
                    const float d = kvq_exact<V>(x[k], c);
                    be[k] = d < bd[k] ? e : be[k];
                    bd[k] = d < bd[k] ? d : bd[k];
                }
            }
#pragma unroll
            for (int k = 0; k < TOK; ++k)
                if (t + k * rows < nt) dst[(size_t)(t + k * rows) * a.P + p] = (uint8_t)be[k];
        }
    } else {
        const int lanes = 1 << a.log_lanes, sub = tid & (lanes - 1), n_items = nt * a.P;
        // (all lanes of a wavefront stay to the end: they merge what they found)
        for (int i0 = 0; i0 < n_items; i0 += 256 >> a.log_lanes) {
            const int i = min(i0 + (tid >> a.log_lanes), n_items - 1), t = i / a.P, p = i - t * a.P;
            const V16 x = kvq_load<V>(xs + (size_t)t * a.D + p * V);
            const half_t *grp = cb + (size_t)(p / a.PG) * (a.E + 1) * V;
            float bd = INFINITY;
            int be = sub;      // (nothing is closer than infinity: entry 0, as the first lane has it)
            for (int e = sub; e < a.E; e += 4 * lanes) {   // (four lookups and distances side by side)
                float d[4];
#pragma unroll
                for (int k = 0; k < 4; ++k)   // (past the end: the last entry, whose own index is smaller)
                    d[k] = kvq_exact<V>(x, kvq_load<V>(grp + (size_t)min(e + k * lanes, a.E - 1) * V));
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    be = d[k] < bd ? e + k * lanes : be;
                    bd = d[k] < bd ? d[k] : bd;
                }
            }
            for (int m = 1; m < lanes; m <<= 1) {   // smaller distance, then smaller index
                const float od = __shfl_xor(bd, m, 64);
                const int oe = __shfl_xor(be, m, 64);
                be = od < bd || (od == bd && oe < be) ? oe : be;
                bd = od < bd ? od : bd;
            }
            if (sub == 0 && i0 + (tid >> a.log_lanes) < n_items) dst[(size_t)t * a.P + p] = (uint8_t)be;
        }
    }
}

// Prompt-sized calls.  The scan above spends 14 vector instructions on every (item, entry) pair; here the matrix cores
// do the pairs and the vector ALU only looks for the minimum.
//   With h_e = |c_e|^2 / 2 the closest entry minimises s_e = h_e - x.c_e (d = |x|^2 + 2 s).  One
//   v_mfma_f32_32x32x16_f16 gives s for 32 entries and 32 items: k = 0 .. V - 1 holds A = -c, B = x (both exact), and
//   k = 8 .. 10 holds h as three halves, scaled by a power of two that B takes back.  Products of two halves are exact in
//   fp32.  E = 256 entries are 8 of these.
//   s is not the definition's distance bit for bit, so it only narrows the search: a lane keeps the minimum of each group
//   of eight entries (the group's number in the four low mantissa bits), the best group and the value of the second best.
//   If the second best is further away than the error of s can bridge, the definition's winner is in the best group, and
//   that is looked at once more: by s in fp32 from |c|^2 / 2, which is enough unless two entries of the group are too close in
//   their turn, or by the definition's distances (smaller index on a tie).  Otherwise -- a near tie between groups, or anything not finite, for which the comparison is
//   false -- the whole codebook is scanned as the definition says.  So the codes are those of the definition, always.
//   Error bound, in units of |x|^2 + |c|max^2, which bounds every |s|, term and partial sum: 17 products and sums to 2^-23
//   each, 15 ulp of the packed bits 2^-19.1, h itself (V + 2) 2^-24 and its split 2^-22: below 2^-17.7; the definition's
//   own rounding, (V + 2) 2^-24 of d / 2, below 2^-20.6.  Two distances are ordered as their s are when these lie more than
//   2^-16.4 apart: 2^-16 is used.  (The split is that good while |c|max^2 lies in [kQuantMinC2, kQuantMaxC2]; outside, every
//   item is scanned.  The matrix cores of this chip take subnormal halves as they are.)
//   (That s: V + 1 roundings to 2^-24 and 15 ulp of packed bits, below 2^-18.4.)
// Bound: vector issue, about 320 instructions per 64 items and wavefront (208 for minima, 32 + 20 for the group) against 16 matrix
// instructions; counters read 370: these 16 with them, and some 30 for the codebooks (450 a wavefront, 16 iterations) and rare paths.  An iteration covers 64 items, so that loads, addresses, norms, the group and the store serve a whole wavefront (the
// minima lie in two lanes per item, and one lane swap brings them to the item's own lane); with 32 items, two lanes each, and the
// group by the definition it was 251 per 32.  B2 H32, 2048 tokens, one codebook per head and side (4.2 M items per side): 112 us with
// 32 items, 92 now, where a scan of every pair took 546.
constexpr int kQuantMfmaTokens = 128;        // tokens per workgroup
// i / PG for the items of a workgroup (i < 128 PG, PG <= 128) by a 24-bit product and a shift: with m = ceil(2^21 / PG) the
// excess i (m PG - 2^21) stays below 2^14 * 2^7 = 2^21, and the product below 2^29.
constexpr unsigned kvq_inverse(int PG) { return ((1u << 21) + PG - 1) / PG; }
constexpr unsigned kvq_quotient(unsigned i, unsigned inverse) { return (i * inverse) >> 21; }
constexpr bool kvq_quotient_exact() {
    for (unsigned PG = 1; PG <= 128; ++PG)
        for (unsigned t = 0; t < 128; ++t)   // (between two multiples the quotient cannot fall)
            if (kvq_quotient(t * PG, kvq_inverse((int)PG)) != t || kvq_quotient(t * PG + PG - 1, kvq_inverse((int)PG)) != t) return false;
    return true;
}
static_assert(kQuantMfmaTokens <= 128 && kvq_quotient_exact(), "");
constexpr float kQuantBound = 1.52587890625e-5f;           // 2^-16
constexpr float kQuantMinC2 = 1e-6f, kQuantMaxC2 = 1e9f;   // (the largest h that 2^15 of headroom takes is 2^30)

// min(a, b) as the median with a minus infinity that the compiler does not see through: one instruction (fminf first
// quiets operands that come straight from a matrix instruction, two more)
__device__ __forceinline__ float min2f(float a, float b, float ninf) { return __builtin_amdgcn_fmed3f(a, b, ninf); }

// The entry with the smaller distance of lanes l and l + 32, whose lower one has the smaller indices.
__device__ __forceinline__ int closer_of_two_lanes(float d, int e) {
    const auto dm = __builtin_amdgcn_permlane32_swap(__float_as_uint(d), __float_as_uint(d), false, false);
    const auto em = __builtin_amdgcn_permlane32_swap((unsigned)e, (unsigned)e, false, false);
    return __uint_as_float(dm[1]) < __uint_as_float(dm[0]) ? (int)em[1] : (int)em[0];
}

// TILES: tiles of 32 entries, 1, 2, 4 or 8, the fewest that hold E; codebooks are padded to that.
// WAY: who looks at the eight entries of the best group.  kKvqPair: the two lanes that hold an item's minima, four each;
// 32 items at a time.  kKvqOwn: 64 items at a time, each lane its own item.  kKvqNorms: the same by s once more, with the entries'
// |c|^2 / 2 from LDS, and by the definition only where two entries of the group are too close (run_kvq_mfma chooses).
enum { kKvqPair, kKvqOwn, kKvqNorms };
template <int V, int TILES, int WAY>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 4))) void kv_quantize_mfma_kernel(KvQuantArgs a) {
    constexpr int EP = 32 * TILES, STEP = WAY == kKvqPair ? 32 : 64;
    constexpr bool NORMS = WAY == kKvqNorms;
    extern __shared__ __align__(16) unsigned char smem[];
    half_t *cb = reinterpret_cast<half_t *>(smem);                                      // [G][EP][V], infinite past E
    float *half_norms = reinterpret_cast<float *>(cb + (size_t)a.G * EP * V);           // [G][EP] |c|^2 / 2 (NORMS)
    float *c2m = half_norms + (NORMS ? (size_t)a.G * EP : 0);                           // [G]  largest |c|^2
    uint8_t *out = reinterpret_cast<uint8_t *>(c2m + ((a.G + 3) & ~3));       // [tokens][P]
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, NW = blockDim.x >> 6;
    const int ln = lane & 31, lh = lane >> 5;
    const int bh = blockIdx.x, h = bh % a.H, side = blockIdx.z;
    const int t0 = blockIdx.y * a.tokens, nt = min(a.tokens, a.n_new - t0);

    const half_t *src = a.cb[side] + (size_t)h * a.G * a.E * V;
    // one wavefront per group of entries: the entries to LDS, the largest |c|^2 by a butterfly
    for (int g = wave; g < a.G; g += NW) {
        float m = 0.f;
        for (int e = lane; e < EP; e += 64) {
            V16 c;
            c.u = make_uint4(0x7C007C00u, 0x7C007C00u, 0x7C007C00u, 0x7C007C00u);
            if (e < a.E) {
                c = kvq_load<V>(src + ((size_t)g * a.E + e) * V);
                float n = 0.f;
#pragma unroll
                for (int k = 0; k < V; ++k) n = __builtin_fmaf((float)c.h8[k], (float)c.h8[k], n);
                // as bits, so that a NaN (above infinity) stays
                m = __uint_as_float(max(__float_as_uint(m), __float_as_uint(n) & 0x7FFFFFFFu));
                if (NORMS) half_norms[g * EP + e] = 0.5f * n;
            }
#pragma unroll
            for (int k = 0; k < V / 2; ++k) reinterpret_cast<uint32_t *>(cb + (size_t)(g * EP + e) * V)[k] = c.w[k];
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1)
            m = __uint_as_float(max(__float_as_uint(m), (unsigned)__shfl_xor((int)__float_as_uint(m), o, 64)));
        if (lane == 0) c2m[g] = m;
    }
    __syncthreads();

    float ninf;
    asm("s_mov_b32 %0, 0xff800000" : "=s"(ninf));
    const unsigned char *xs = reinterpret_cast<const unsigned char *>(a.x[side] + ((size_t)bh * a.n_new + t0) * a.D);
    const int n_items = nt * a.PG, n_ct = (n_items + STEP - 1) / STEP;   // per group
    const int R = max(1, NW / a.G);                              // wavefronts that share a group
    for (int u = wave; u < a.G * R; u += NW) {
        const int g = u / R;
        const half_t *cbg = cb + (size_t)g * EP * V;
        const float c2 = c2m[g];
        const bool in_range = c2 >= kQuantMinC2 && c2 <= kQuantMaxC2;
        // h = 2^-k (h1 + h2 + h3) with the largest h just below 2^15 (k within what a half can take back)
        const int k = min(max(15 - (int)((__float_as_uint(0.5f * c2) >> 23) & 255) + 126, -15), 24);
        const float up = __uint_as_float((unsigned)(127 + k) << 23);
        const half_t down = (half_t)__uint_as_float((unsigned)(127 - k) << 23);
        // the codebook of the group as matrix operands: entry 32 t + ln.  Past E: the first entry of the same group of eight
        // once more, which changes no minimum, or the last entry (groups without entries, and all of nearly 256: an item whose
        // closest entry is the last one then ties and is scanned, but the select, once per workgroup and tile, costs more)
        half8_t A[TILES];
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
            const int e = 32 * t + ln, last = a.E - 1;
            const V16 c = kvq_load<V>(cbg + (TILES < 8 && e > last ? min(32 * t + (ln & 20), last) : min(e, last)) * V);
            float hh = 0.f;
#pragma unroll
            for (int i = 0; i < V; ++i) hh = __builtin_fmaf((float)c.h8[i], (float)c.h8[i], hh);
            hh *= 0.5f * up;
            const half_t h1 = (half_t)hh;
            const half_t h2 = (half_t)(hh - (float)h1);
            const half_t h3 = (half_t)((hh - (float)h1) - (float)h2);
            V16 v;
            const half2_t h12 = {h1, h2}, h30 = {h3, (half_t)0.f};
#pragma unroll
            for (int i = 0; i < 4; ++i) v.w[i] = lh ? 0u : i < V / 2 ? c.w[i] ^ 0x80008000u : 0u;
            if (lh) {
                v.h2[0] = h12;
                v.h2[1] = h30;
            }
            A[t] = v.h8;
        }
        // operand words of the upper half's k: what takes the power of two of h back
        const half2_t dd = {down, down}, d0 = {down, (half_t)0.f};
        const unsigned back[4] = {__builtin_bit_cast(unsigned, dd), __builtin_bit_cast(unsigned, d0), 0u, 0u};
        const float bound_c2 = kQuantBound * c2;
        auto item_off = [&](unsigned i) {   // index of the sub-vector in [token][P]
            return __umul24(__umul24(i, a.pg_inverse) >> 21, (unsigned)(a.P - a.PG)) + i + (unsigned)(g * a.PG);   // (kvq_quotient)
        };
        auto lane_off = [&](int ct) { return item_off((unsigned)min(ct * STEP + lane % STEP, n_items - 1)); };
        auto load_item = [&](unsigned off) { return kvq_load<V>(xs + off * (V * 2)); };
        unsigned off = lane_off(min(u % R, n_ct - 1));
        V16 xb = load_item(off);
        for (int ct = u % R; ct < n_ct; ct += R) {
            const unsigned off_next = lane_off(min(ct + R, n_ct - 1));
            const V16 xnext = load_item(off_next);
            V16 bop[2];   // items 0 .. 31 and 32 .. 63
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const auto r = __builtin_amdgcn_permlane32_swap(i < V / 2 ? xb.w[i] : 0u, back[i], false, false);
                bop[0].w[i] = r[0];
                bop[1].w[i] = r[1];
            }
            const float16_t zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            float best[2] = {INFINITY, INFINITY}, second[2] = {INFINITY, INFINITY};
            auto minima = [&](const half8_t &items, float &lowest, float &next) {
                float16_t s = __builtin_amdgcn_mfma_f32_32x32x16_f16(A[0], items, zero, 0, 0, 0);
#pragma unroll
                for (int t = 0; t < TILES; ++t) {
                    float16_t sn = s;   // the next tile's products run while this tile's minima are taken
                    if (t + 1 < TILES) sn = __builtin_amdgcn_mfma_f32_32x32x16_f16(A[t + 1 < TILES ? t + 1 : 0], items, zero, 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    float key[2];
#pragma unroll
                    for (int hf = 0; hf < 2; ++hf) {
                        float m = min2f(s[8 * hf], s[8 * hf + 1], ninf);
                        m = fminf(fminf(m, s[8 * hf + 2]), s[8 * hf + 3]);
                        m = fminf(fminf(m, s[8 * hf + 4]), s[8 * hf + 5]);
                        m = fminf(fminf(m, s[8 * hf + 6]), s[8 * hf + 7]);
                        key[hf] = __uint_as_float((__float_as_uint(m) & 0xFFFFFFF0u) | (unsigned)(2 * t + hf));
                        // (a group whose first row, 16 hf + 4 lh, is past E has no entries and is never the closest; of 256 or
                        // nearly 256 the few such groups may tie with the last entry instead, which is cheaper)
                        if (TILES < 8) key[hf] = 32 * t + 16 * hf + 4 * lh < a.E ? key[hf] : 3e38f;
                    }
                    // second best of {lowest <= next, two keys}
                    next = min2f(next, __builtin_amdgcn_fmed3f(lowest, key[0], key[1]), ninf);
                    lowest = fminf(fminf(lowest, key[0]), key[1]);
                    s = sn;
                }
            };
            minima(bop[0].h8, best[0], second[0]);
            asm volatile("" : "+v"(best[0]), "+v"(second[0]));   // (or the compiler moves the minima behind the branch, and all products lie in scratch)
            if (STEP == 64 && ct * 64 + 32 < n_items) minima(bop[1].h8, best[1], second[1]);
            // an item's entries lie in two lanes, 32 apart: both lanes' values to the item's own lane, or to both
            const auto bm = __builtin_amdgcn_permlane32_swap(__float_as_uint(best[0]), __float_as_uint(best[STEP / 64]), false, false);
            const auto sm = __builtin_amdgcn_permlane32_swap(__float_as_uint(second[0]), __float_as_uint(second[STEP / 64]), false, false);
            const float bl = __uint_as_float(bm[0]), bu = __uint_as_float(bm[1]);
            const float win = min2f(bl, bu, ninf);
            const float runner_up = fminf(fmaxf(bl, bu), fminf(__uint_as_float(sm[0]), __uint_as_float(sm[1])));
            float x2 = 0.f;
#pragma unroll
            for (int i = 0; i < V; ++i) x2 = __builtin_fmaf((float)xb.h8[i], (float)xb.h8[i], x2);
            const float bound = __builtin_fmaf(kQuantBound, x2, bound_c2);
            const bool live = lane < STEP && ct * STEP + lane < n_items;
            const bool sure = runner_up - win > bound && in_range;
            // entries of the group: rows 16 (grp & 1) + 4 (half whose lane holds them) + {0 .. 3, 8 .. 11} of tile grp / 2
            const int e0 = 16 * (int)(__float_as_uint(win) & (2u * TILES - 1u)) + (bu < bl ? 4 : 0);
            int be = e0;
            bool within = false;   // the group's closest entry is known
            if constexpr (NORMS) {
                const float *hg = half_norms + g * EP + e0;
                float lowest = INFINITY, next = INFINITY;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const float4_t h4 = *reinterpret_cast<const float4_t *>(hg + 8 * q);
                    V16 c4[V / 2];   // four entries
#pragma unroll
                    for (int i = 0; i < V / 2; ++i) c4[i] = ld16(cbg + (size_t)(e0 + 8 * q) * V + 8 * i);
                    float key[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        float d = h4[j];
#pragma unroll
                        for (int i = 0; i < V; ++i) d = __builtin_fmaf(-(float)xb.h8[i], (float)c4[(j * V + i) / 8].h8[(j * V + i) % 8], d);
                        key[j] = __uint_as_float((__float_as_uint(d) & 0xFFFFFFF0u) | (unsigned)(8 * q + j));
                    }
#pragma unroll
                    for (int j = 0; j < 4; j += 2) {
                        next = min2f(next, __builtin_amdgcn_fmed3f(lowest, key[j], key[j + 1]), ninf);
                        lowest = fminf(fminf(lowest, key[j]), key[j + 1]);
                    }
                }
                within = next - lowest > bound;
                be = e0 + (int)(__float_as_uint(lowest) & 15u);
            }
            if (!NORMS || __ballot(sure && !within && live)) {
                const int first = WAY == kKvqPair ? e0 + 8 * lh : e0;
                float bd = kvq_exact<V>(xb, kvq_load<V>(cbg + (size_t)first * V));
                int ge = first;
#pragma unroll
                for (int i = 1; i < (WAY == kKvqPair ? 4 : 8); ++i) {
                    const int e = first + i + (i & 4);
                    const float d = kvq_exact<V>(xb, kvq_load<V>(cbg + (size_t)e * V));
                    ge = d < bd ? e : ge;
                    bd = d < bd ? d : bd;
                }
                if (WAY == kKvqPair) ge = closer_of_two_lanes(bd, ge);
                be = within ? be : ge;
            }
            unsigned long long left = __ballot(!sure && live);
            if (left) {
                if (__popcll(left) > STEP * 3 / 8) {
                    // many: every lane scans the entries for its item, two lanes one half each
                    const int from = WAY == kKvqPair ? lh * 128 : 0, to = WAY == kKvqPair ? min(from + 128, a.E) : a.E;
                    float bd2 = INFINITY;
                    int be2 = from;
                    for (int e = from; e < to; ++e) {
                        const float d = kvq_exact<V>(xb, kvq_load<V>(cbg + (size_t)e * V));
                        be2 = d < bd2 ? e : be2;
                        bd2 = d < bd2 ? d : bd2;
                    }
                    if (WAY == kKvqPair) be2 = closer_of_two_lanes(bd2, be2);
                    be = sure ? be : be2;
                } else {
                    // few: one after the other, the 64 lanes taking the entries in turn
                    for (; left; left &= left - 1) {
                        const int j = __ffsll((long long)left) - 1;
                        V16 xj;
                        xj.u = make_uint4(0, 0, 0, 0);
#pragma unroll
                        for (int q = 0; q < V / 2; ++q) xj.w[q] = (unsigned)__builtin_amdgcn_readlane((int)xb.w[q], j);
                        float bd2 = INFINITY;
                        int be2 = lane;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {   // (entries past E are infinitely far)
                            if (64 * q >= EP) break;
                            const float d = kvq_exact<V>(xj, kvq_load<V>(cbg + (size_t)min(lane + 64 * q, EP - 1) * V));
                            be2 = d < bd2 ? lane + 64 * q : be2;
                            bd2 = d < bd2 ? d : bd2;
                        }
                        const int code = kvq_wave_argmin(bd2, be2);
                        be = lane == j ? code : be;
                    }
                }
            }
            if (live) out[off] = (uint8_t)be;
            xb = xnext;
            off = off_next;
        }
    }
    __syncthreads();
    uint8_t *dst = a.codes[side] + ((size_t)bh * a.T + a.pos + t0) * a.P;
    if ((a.P & 3) == 0) {
        for (int i = tid; i < nt * a.P / 4; i += blockDim.x)
            reinterpret_cast<uint32_t *>(dst)[i] = reinterpret_cast<const uint32_t *>(out)[i];
    } else {
        for (int i = tid; i < nt * a.P; i += blockDim.x) dst[i] = out[i];
    }
}

enum { kKvqScan, kKvqLane, kKvqMfma };
constexpr int kQuantScanTokens = 16, kQuantLaneTokens = 128;   // tokens per workgroup, at most
constexpr int kQuantLaneBytes = 16 * 1024;                     // of codebooks: more leave a CU too few wavefronts

namespace {

int ceil_div(long a, long b) { return (int)((a + b - 1) / b); }
// Tokens per workgroup of the matrix-core kernel: as many as leave the chip two rounds of workgroups (a workgroup stages its
// codebooks first).
int kvq_mfma_tokens(int bh, int n_new) {
    int tokens = kQuantMfmaTokens;
    while (tokens > 16 && (long)bh * 2 * ceil_div(n_new, tokens) < 1024) tokens /= 2;
    return tokens;
}
// Lanes that share an item: as many as give 256 lanes work.
int kvq_log_lanes(int items) {
    int log_lanes = 0;
    while (log_lanes < 6 && items << (log_lanes + 1) <= 256) ++log_lanes;
    return log_lanes;
}
// Four tokens at a time save three of four lookups of an entry (v = 8 is bound by its distances: 8 entries 27.1 us with one,
// 28.0 with four; v = 4 34.3 / 30.3).
bool kvq_four_tokens(int P, int v, int n_new) { return v <= 4 && n_new >= 4 * (256 / P); }

// Workgroups of the scan that share the items of a token range, up to four: a wavefront takes its groups and items one after the other,
// each a trip to memory or a reduction, so few sequences are spread over the chip.  32 codebooks of v = 4 per head and side,
// H32, one token: B1 5.0 -> 3.0 us, B3 5.0 -> 4.4, four tokens 10.7 -> 7.3; beyond 768 workgroups only long chains gain (B8, one
// token 6.6 / 6.7; 64 codebooks of v = 2, six tokens 34.5 -> 29.3).  Fewer than 32 items a workgroup: not where that makes 257 to 512
// workgroups, which take 5 % longer than half as many of twice the items (88 sequence-heads, 16 items 3.18 / 3.47); up to 256 take 18 % less,
// 513 to 768 2 to 9 % (96 sequence-heads, 32 items of 32 groups 4.3 -> 4.1 with four).
int kvq_share(long bh, int ranges, int items) {
    int share = 1;
    for (; share < 4 && 16 * share <= items; share *= 2) {
        const long wgs = bh * 4 * ranges * share;   // with twice the share
        if (wgs > (items >= 128 * share ? 1024 : 768) || (items < 32 * share && wgs > 256 && wgs <= 512)) break;
    }
    return share;
}

// The kernel with the least estimated time (us): the chain of one workgroup or the instructions of all of them (a vector
// instruction of a wavefront: 1.63e-6 us of the chip), whichever is longer.  Over 10815 measured calls (B 1 .. 64, 1 to
// 2048 tokens, 8 to 256 entries, 1 to 64 groups, head sizes 64 to 256) the pick takes 1.5 % more than the best of the three on
// average and 25 % or more in the worst hundredth (6 % and 80 % while the scan counted as if no workgroups shared it).  Some,
// us, scan / lane / matrix cores: one group of 256, v = 4, one token, B4 4.3 / 4.1 / 4.8,
// B16 8.6 / 6.3 / 5.4, B64 25.2 / 16.8 / 15.9; 32 groups of 256, B4, 4 tokens 11.0 / - / 14.3, 22 sequence-heads, 6 tokens 5.1 / - / 13.4, 4, 10 tokens 6.6 / - / 13.1;
// 8 groups of 64, B16, one token 8.6 / 4.0 / 6.7; 16 entries, v = 4, B64, 4 tokens 73 / 7.2 / 11.1, B2, 2048 tokens 1052 / 51 / 43.
// Workgroups that share a chain are in each other's way: it takes up to 1.7 times what its part of the items would, and longer the more
// instructions there are (without that, 104 sequence-heads, 15 tokens, 64 groups of 128, v = 2 came to the scan, 33.0 / - / 24.5).
int kvq_choice(int bh, int P, int v, int E, int G, int n_new) {
    const double kInst = 1.63e-6;
    double best = 1e300;
    int pick = kKvqScan;
    auto consider = [&](int kernel, double chain, double wgs, double start, double inst) {
        const double t = std::max(chain, wgs * (start + inst * kInst));
        if (t < best) {
            best = t;
            pick = kernel;
        }
    };
    const double sides = 2.0 * bh;
    {   // a wavefront takes one item after the other
        const int tokens = std::min(n_new, kQuantScanTokens), items = tokens * P, ranges = ceil_div(n_new, tokens), share = kvq_share(bh, ranges, items);
        const double item = 0.33 + 0.045 * v, inst = items * (52.0 + 9 * v);
        double chain = ceil_div(items, 8) * item;
        if (share > 1) chain = std::min(chain, 1.6 * ceil_div(items, 8 * share) * item + 0.5 * sides * ranges * inst * kInst);
        consider(kKvqScan, chain, sides * ranges, 0.0022 * share, inst);
    }
    if (G * E * v * 2 <= kQuantLaneBytes) {
        const int tokens = std::min(n_new, kQuantLaneTokens), items = tokens * P, log_lanes = kvq_log_lanes(items);
        const bool four = kvq_four_tokens(P, v, n_new);
        const int entries = ceil_div(E, 1 << log_lanes);
        const int waves = four ? 16 * ceil_div(tokens, 4 * (256 / P)) : ceil_div((long)items << log_lanes, 64);
        const double per_entry = four ? 1 + 2.7 * v : 4 + 2.5 * v;
        consider(kKvqLane, ceil_div(waves, 4) * (entries * (0.03 + 0.005 * v) + 0.06 * log_lanes) + 5e-5 * (G * E * v * 2), sides * ceil_div(n_new, tokens), 0.0015,
                 waves * (entries * per_entry + 12 * log_lanes) + G * E * 0.4);
    }
    {
        const int tiles = E <= 32 ? 1 : E <= 64 ? 2 : E <= 128 ? 4 : 8, most = kvq_mfma_tokens(bh, n_new), tokens = std::min(n_new, most);
        const int items = tokens * (P / G), columns = ceil_div(items, 32);   // per group; column tiles of 32 items
        const int waves = 4 * ((long)G * 64 * tiles * v + tokens * P) > 160 * 1024 ? 8 : 4, share = std::max(1, waves / G);
        const double chain = ceil_div(G, waves) * (0.6 + 0.2 * tiles + 0.08 * v + (ceil_div(columns, share) - 1) * (0.5 + 0.06 * tiles));
        consider(kKvqMfma, chain + 1.8e-5 * (G * E * v * 2), sides * ceil_div(n_new, most), 0.0022,
                 G * (40.0 + 36 * tiles + columns * 14.0 * tiles + (items <= 32 * share ? columns * 95.0 : ceil_div(items, 64) * (110.0 + 14 * v))));
    }
    return pick;
}

}  // namespace

int kv_quantize_kernel_of(const vq_kv_t *kv, int n_new) {
    return kvq_choice(kv->B * kv->H, kv->D / kv->v, kv->v, kv->n_entries, kv->cb_groups, n_new);
}

namespace {

// A launch of the matrix-core kernel.
struct KvqMfmaPlan {
    int tokens, threads, way;
    size_t lds;
};
KvqMfmaPlan kvq_mfma_plan(int bh, int P, int v, int E, int G, int n_new) {
    const int tiles = E <= 32 ? 1 : E <= 64 ? 2 : E <= 128 ? 4 : 8;
    KvqMfmaPlan p;
    p.tokens = kvq_mfma_tokens(bh, n_new);
    p.lds = (size_t)G * 32 * tiles * v * sizeof(half_t) + (((size_t)G + 3) & ~(size_t)3) * 4 + (size_t)p.tokens * P;
    // a CU holds 16 wavefronts of this kernel: two workgroups of 8 where 64 KiB of codebooks are staged, four of 4 otherwise
    p.threads = 4 * p.lds > 160 * 1024 ? 512 : 256;
    // Two lanes per item where a wavefront has 32 items of a group or fewer (12 tokens of 8 groups ...): 64 at a time leave half of
    // the lanes idle.  And where a call is as long as one wavefront's chain (up to two workgroups a CU) and units of 32 spread
    // better over the wavefronts: an iteration over 64 takes 1.7 times as long.
    const int items = std::min(p.tokens, n_new) * (P / G), share = std::max(1, p.threads / 64 / G);
    const int by_32 = ceil_div(ceil_div(items, 32), share), by_64 = ceil_div(ceil_div(items, 64), share);
    const bool chain = (long)bh * 2 * ceil_div(n_new, p.tokens) <= 512;
    // the norms, where they do not cost a workgroup per CU and no group is in part past the last entry
    const size_t with_norms = p.lds + (size_t)G * 32 * tiles * sizeof(float);
    if (items <= 32 * share || (chain && 10 * by_32 < 17 * by_64)) {
        p.way = kKvqPair;
    } else if (E % 16 == 0 && with_norms * (p.threads == 512 ? 2 : 4) <= 160 * 1024) {
        p.way = kKvqNorms;
        p.lds = with_norms;
    } else {
        p.way = kKvqOwn;
    }
    return p;
}

template <int V, int TILES, int WAY>
int run_kvq_mfma_as(const KvQuantArgs &a, int bh, const KvqMfmaPlan &p, hipStream_t s) {
    static KernelSetup setup;
    if (int st = kernel_setup(reinterpret_cast<const void *>(&kv_quantize_mfma_kernel<V, TILES, WAY>), p.lds, false, setup)) return st;
    kv_quantize_mfma_kernel<V, TILES, WAY><<<dim3(bh, (a.n_new + a.tokens - 1) / a.tokens, 2), p.threads, p.lds, s>>>(a);
    return launch_status();
}

template <int V, int TILES>
int run_kvq_mfma(const KvQuantArgs &a, int bh, const KvqMfmaPlan &p, hipStream_t s) {
    if (p.way == kKvqPair) return run_kvq_mfma_as<V, TILES, kKvqPair>(a, bh, p, s);
    if (p.way == kKvqNorms) return run_kvq_mfma_as<V, TILES, kKvqNorms>(a, bh, p, s);
    return run_kvq_mfma_as<V, TILES, kKvqOwn>(a, bh, p, s);
}

template <int V>
int run_kvq_lane(KvQuantArgs &a, int bh, hipStream_t s) {
    a.tokens = std::min(a.n_new, kQuantLaneTokens);
    a.log_lanes = kvq_log_lanes(a.tokens * a.P);
    const dim3 grid(bh, (a.n_new + a.tokens - 1) / a.tokens, 2);
    const size_t lds = (size_t)a.G * (a.E + 1) * V * sizeof(half_t);   // (below 64 KiB: kQuantLaneBytes)
    if constexpr (V <= 4)
        if (kvq_four_tokens(a.P, V, a.n_new)) {
            kv_quantize_lane_kernel<V, 4><<<grid, 256, lds, s>>>(a);
            return launch_status();
        }
    kv_quantize_lane_kernel<V, 1><<<grid, 256, lds, s>>>(a);
    return launch_status();
}

template <int V>
int run_kvq(KvQuantArgs &a, int bh, hipStream_t s) {
    const int kernel = kvq_choice(bh, a.P, V, a.E, a.G, a.n_new);
    if (kernel == kKvqLane) return run_kvq_lane<V>(a, bh, s);
    if (kernel == kKvqScan) {
        a.tokens = std::min(a.n_new, kQuantScanTokens);
        const int ranges = ceil_div(a.n_new, a.tokens);
        a.share = kvq_share(bh, ranges, a.tokens * a.P);
        if (a.share > 1)
            kv_quantize_scan_kernel<V, true><<<dim3(bh, ranges, 2 * a.share), 512, 0, s>>>(a);
        else
            kv_quantize_scan_kernel<V, false><<<dim3(bh, ranges, 2), 512, 0, s>>>(a);
        return launch_status();
    }
    a.pg_inverse = kvq_inverse(a.PG);
    const KvqMfmaPlan p = kvq_mfma_plan(bh, a.P, V, a.E, a.G, a.n_new);
    a.tokens = p.tokens;
    if (a.E <= 32) return run_kvq_mfma<V, 1>(a, bh, p, s);
    if (a.E <= 64) return run_kvq_mfma<V, 2>(a, bh, p, s);
    if (a.E <= 128) return run_kvq_mfma<V, 4>(a, bh, p, s);
    return run_kvq_mfma<V, 8>(a, bh, p, s);
}

}  // namespace

// What a call does (for tests): kernel, its variant (matrix cores), tokens per workgroup, threads, workgroups that share a token range.
void kv_quantize_plan_of(const vq_kv_t *kv, int n_new, int out[5]) {
    const int bh = kv->B * kv->H, P = kv->D / kv->v;
    out[0] = kv_quantize_kernel_of(kv, n_new);
    out[1] = 0;
    out[2] = std::min(n_new, out[0] == kKvqScan ? kQuantScanTokens : kQuantLaneTokens);
    out[3] = out[0] == kKvqScan ? 512 : 256;
    out[4] = out[0] == kKvqScan ? kvq_share(bh, ceil_div(n_new, out[2]), out[2] * P) : 1;
    if (out[0] == kKvqMfma) {
        const KvqMfmaPlan p = kvq_mfma_plan(bh, P, kv->v, kv->n_entries, kv->cb_groups, n_new);
        out[1] = p.way;
        out[2] = p.tokens;
        out[3] = p.threads;
    }
}

int launch_kv_quantize(const vq_kv_t *kv, const void *k_new, const void *v_new, int n_new, int pos, hipStream_t s) {
    const size_t cb_bytes = (size_t)kv->cb_groups * kv->n_entries * kv->v * sizeof(half_t);
    if (cb_bytes > 64 * 1024 || cb_bytes % 16 != 0) return VQ_ERR_UNSUPPORTED;
    KvQuantArgs a;
    a.x[0] = (const half_t *)k_new;
    a.x[1] = (const half_t *)v_new;
    a.cb[0] = (const half_t *)kv->k_codebooks;
    a.cb[1] = (const half_t *)kv->v_codebooks;
    a.codes[0] = (uint8_t *)const_cast<void *>(kv->k_codes);
    a.codes[1] = (uint8_t *)const_cast<void *>(kv->v_codes);
    a.H = kv->H;
    a.T = kv->T;
    a.D = kv->D;
    a.P = kv->D / kv->v;
    a.E = kv->n_entries;
    a.G = kv->cb_groups;
    a.n_new = n_new;
    a.pos = pos;
    a.PG = a.P / a.G;
    a.pg_inverse = 0;
    const int bh = kv->B * kv->H;
    if (kv->v == 8) return run_kvq<8>(a, bh, s);
    if (kv->v == 4) return run_kvq<4>(a, bh, s);
    return run_kvq<2>(a, bh, s);
}

}  // namespace vq
