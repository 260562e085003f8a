// Products of a VQ weight with a few to a few hundred tokens in ONE pass over the codes, on the matrix cores of gfx950:
// vq_gemm for 17 .. 256 tokens and more where the product is small, vq_gemv for several tokens of a codebook that does
// not fit LDS and for nearly 16 of one that does.
// Operation: VQ-LLM (arXiv 2503.02236) Sec. III-C; dequantization of Sec. II-A in front of the matrix instruction.
//
// What bounds it: every workgroup reads its share of X from L2 (41 bytes per clock and CU) and looks up one entry per
// code, from LDS (5.5 per clock and CU) or, for a 2^16-entry codebook, from L2 (0.44).  A workgroup owns 16 RT weight
// rows x 16 CT tokens; each of its wavefronts computes that whole tile over its own part of K, so inside a workgroup
// nothing is looked up or read twice, no barrier stands in the main loop, and the partial tiles meet in LDS once at
// the end.  16 RT trades X traffic (N / 16 RT workgroups read all of X), 16 CT lookups (M / 16 CT workgroups look up
// the same codes): skinny_tile() weighs the two.
//
// Operands: v_mfma_f32_16x16x32_f16, A = 16 weight rows (a lane's operand is 8 consecutive k of its row = one v = 8
// entry or two v = 4 entries, straight from the codebook), B = 16 tokens.  Both want lane l to hold row l % 16, which is
// the worst order for a load: neighbouring lanes on different lines, 16 bytes of each (measured: 13 bytes of X per clock
// and CU, however deep the prefetch).  So X is loaded as whole contiguous pieces of token rows (8 lanes a line), written
// to a small LDS area of the wavefront's own and read back as operands: N = K = 4096, two codebooks, 77 tokens 21.2 ->
// 13.0 us, 256 tokens 25.2 -> 18.4.  A lane loads 16 bytes of codes, the four lanes of a row 64 consecutive bytes; a
// 4 x 4 transposition of the dwords over the four lanes (v_permlane32_swap, v_permlane16_swap) gives step i the i-th 16
// bytes of the 64, one dword per lane, which makes the X of a step contiguous.
//
// Measured (N = K = 4096 unless said; before: 16 tokens a launch from LDS codebooks, a 256-token tile from L2 ones):
// two 256-entry codebooks, 77 tokens 37.8 -> 12.9 us, 256 tokens 120 -> 18.6; 12-bit codes, 77 tokens 40.8 -> 15.4; 2^16
// entries, 32 tokens 160 -> 14.7, 256 tokens 175 -> 32; N = 11008, 8 tokens 62.5 -> 30.5 (two passes of gathers before,
// one now: 0.37 per clock and CU).
#include <algorithm>
#include <type_traits>

#include "vq_common.h"

namespace vq {

namespace {

typedef float float4v_t __attribute__((ext_vector_type(4)));

struct SkinnyArgs {
    const void *codes;
    const half_t *cb, *scale, *x;
    half_t *y;
    int N, K, M, E;
    int ops;   // MFMA operands (8 consecutive k) per row
    int nit;   // wavefront iterations over K
    int tiles_k, tile_ops, tile_n;   // per-tile codebooks: sets per row of tiles, operands per tile, rows per tile (0: per tensor)
    int groups_m;                    // workgroups along the tokens
};

// Code load of a lane and iteration: 16 bytes, 8 for single uint8 codes (rows are multiples of 8 bytes only), 12-byte
// words of 8 codes for packed 12-bit codes.
template <typename CodeT, int V, int R>
struct SkinnyShape {
    static constexpr int BITS = (int)sizeof(CodeT) * 8;
    static constexpr int LB = R * (int)sizeof(CodeT) == 1 ? 8 : 16;
};
template <int V, int R>
struct SkinnyShape<Code12, V, R> {
    static constexpr int BITS = 12;
    static constexpr int LB = 12;
};

// Code number q (static) of the lane's code words.
template <typename CodeT>
__device__ __forceinline__ unsigned skinny_code(const V16 &cd, int q) {
    return sizeof(CodeT) == 1 ? (cd.w[q >> 2] >> (8 * (q & 3))) & 0xFFu : (cd.w[q >> 1] >> (16 * (q & 1))) & 0xFFFFu;
}
template <>
__device__ __forceinline__ unsigned skinny_code<Code12>(const V16 &cd, int q) {
    const int bit = 12 * q, wi = bit >> 5, sh = bit & 31;
    unsigned v = cd.w[wi] >> sh;
    if (sh > 20) v |= cd.w[wi + 1] << (32 - sh);
    return v & 0xFFFu;
}

__device__ __forceinline__ void swap32(uint32_t &a, uint32_t &b) {   // upper half of a <-> lower half of b
    const auto t = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = t[0];
    b = t[1];
}
__device__ __forceinline__ void swap16(uint32_t &a, uint32_t &b) {   // odd rows of 16 lanes of a <-> even rows of b
    const auto t = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = t[0];
    b = t[1];
}

constexpr int skinny_max_waves(bool l2, int rt, int ct) { return !l2 && rt * ct <= 2 ? 16 : 8; }

// Operands of an X unit: two (a line of 128 bytes per token where a lane's operands of a step are one or two), four where a
// step has four or eight.  All eight of one 12-bit codebook would be 456 bytes of scratch per lane (N = K = 4096, 17 / 77 / 256
// tokens 46.9 / 33.7 / 65.9 us, with four 12.2 / 16.8 / 31.4).  With four the {1, 2} tiles and {4, 4} spill up to ten loop
// constants: units of two (K = 11008, 32 tokens 14.6 -> 18.3) or constants formed again for every unit (two 12-bit
// codebooks, 32 tokens 8.3 -> 10.5) spill none and take longer.
constexpr int skinny_unit(int mpi, int opd) { return opd > 2 ? 4 : mpi < 2 ? mpi : 2; }
// Units in flight: up to 64 registers (32 where the accumulators or 16 wavefronts take the rest), a divisor of the
// units per iteration.
constexpr int skinny_depth(int epi, int u, bool l2, int rt, int ct) {
    int d = (rt * ct >= 16 || skinny_max_waves(l2, rt, ct) == 16 ? 8 : 16) / u;
    while (epi % d) --d;
    return d;
}

// L2CB: entries are gathered from global memory (L2); otherwise the codebooks are staged in LDS.
template <typename CodeT, int V, int R, bool L2CB, int RT, int CT>
__global__ __launch_bounds__(64 * skinny_max_waves(L2CB, RT, CT)) void gemm_skinny_kernel(SkinnyArgs a) {
    constexpr int BITS = SkinnyShape<CodeT, V, R>::BITS, LB = SkinnyShape<CodeT, V, R>::LB;
    constexpr int CPO = 8 / V;                         // entries side by side in an operand
    constexpr int MPI = LB * 8 / (BITS * R * CPO);     // operands per lane and iteration
    static_assert(MPI * BITS * R * CPO == LB * 8, "whole operands per code load");
    static_assert(R <= 2, "operands are summed in fp16 (one rounding)");
    constexpr bool TR = LB != 12 && BITS * R * CPO <= 32;   // whole operands per dword: transpose
    constexpr int NS = TR ? LB / 4 : 1, OPD = MPI / NS;     // steps per iteration, operands per step
    // X goes through LDS in units of U operands (32 U k) x 16 tokens, private to the wavefront.  D units per lane are
    // in flight in registers.
    constexpr int U = skinny_unit(MPI, OPD), NU = MPI / U, SEGS = 4 * U, EPI = NU * CT;
    constexpr int D = skinny_depth(EPI, U, L2CB, RT, CT);
    static_assert(D <= EPI && MPI % U == 0 && EPI % D == 0 && (!L2CB || NU % 2 == 0), "slots are the same in every iteration");

    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, nwaves = blockDim.x >> 6;
    const int r = lane & 15, g = lane >> 4;
    const int n0 = (blockIdx.x / a.groups_m) * 16 * RT, m0 = (blockIdx.x % a.groups_m) * 16 * CT;
    const int row_bytes = a.ops * CPO * R * BITS / 8;
    const int slot = !TR || NS == 4 ? g : ((g & 1) << 1) | (g >> 1);   // (two dwords: one swap, lanes 1 and 2 of a row change places)

    const unsigned char *cbase = reinterpret_cast<const unsigned char *>(a.codes) + (size_t)n0 * row_bytes;
    uint32_t crow[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t)   // rows past the end are computed and dropped
        crow[t] = (uint32_t)(min(n0 + 16 * t + r, a.N - 1) - n0) * (uint32_t)row_bytes;
    // X loads: instruction j of a unit covers 64 / SEGS tokens, whole contiguous rows of SEGS 16-byte segments
    const int xseg = lane % SEGS, xtok = lane / SEGS;
    uint32_t xrow[CT][U];   // byte offsets (kSkinnyMaxX)
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int j = 0; j < U; ++j) xrow[c][j] = (uint32_t)min(m0 + 16 * c + j * (64 / SEGS) + xtok, a.M - 1) * (uint32_t)(a.K * 2);

    // Loads carry no condition: a lane past the end of its row reads the row's last bytes, and what it makes of them
    // is zeroed (both operands: an infinity there must not meet a zero).
    auto load_codes = [&](int it, int t, V16 &cd) {
        const unsigned char *p = cbase + (crow[t] + (uint32_t)min((it * 4 + g) * LB, row_bytes - LB));
        if (LB == 16) {
            cd = ld16(p);
        } else if (LB == 12) {
            const uint32_t *c3 = reinterpret_cast<const uint32_t *>(p);
            cd.w[0] = c3[0];
            cd.w[1] = c3[1];
            cd.w[2] = c3[2];
            cd.w[3] = 0;
        } else {
            const V8 c8 = ld8(p);
            cd.w[0] = c8.w[0];
            cd.w[1] = c8.w[1];
            cd.w[2] = cd.w[3] = 0;
        }
    };
    auto transpose = [&](V16 &cd) {
        if (TR && NS == 4) {
            swap32(cd.w[0], cd.w[2]);
            swap32(cd.w[1], cd.w[3]);
            swap16(cd.w[0], cd.w[1]);
            swap16(cd.w[2], cd.w[3]);
        } else if (TR && NS == 2) {
            swap32(cd.w[0], cd.w[1]);
        }
    };
    // position (in operands) of this lane's operand o of an iteration
    auto op_index = [&](int it, int o) { return it * 4 * MPI + ((o / OPD) * 4 + slot) * OPD + o % OPD; };
    const int cb_bytes = L2CB ? 0 : (R * a.E * V * 2 * a.tiles_k + 15) & ~15;
    unsigned char *stage = smem + cb_bytes + wave * (U * 1024);
    // slot of 16-byte segment `seg` of token `tok` of a unit: the 16 tokens of a pass over the banks get different ones
    auto stage_off = [&](int tok, int seg) {
        const int swz = U == 2 ? (tok ^ (tok >> 3)) & 7 : tok & (SEGS < 16 ? SEGS - 1 : 15);
        return tok * (SEGS * 16) + ((seg ^ swz) << 4);
    };
    // A unit is whole steps of the four lanes of a row (their operands lie side by side), or a part of one step (U of the OPD
    // operands of each of the four lanes).
    constexpr bool PART = U < OPD;
    static_assert(PART ? OPD % U == 0 : U % OPD == 0, "units and steps");
    const int xlane = PART ? (xseg / U) * OPD + xseg % U : xseg;
    auto load_x = [&](int it, int e, V16 (&xb)[U]) {   // unit e / CT, token tile e % CT
        const int u = e / CT, first = PART ? u * U / OPD * (4 * OPD) + u * U % OPD : u * SEGS;
        const uint32_t k = min(it * (4 * MPI) + first + xlane, a.ops - 1) * 16;
#pragma unroll
        for (int j = 0; j < U; ++j) xb[j] = ld16(reinterpret_cast<const unsigned char *>(a.x) + (xrow[e % CT][j] + k));
    };
    // registers -> LDS -> operands (a wavefront's LDS operations are carried out in order: one buffer is enough)
    auto stage_x = [&](const V16 (&xb)[U], half8_t (&xo)[U]) {
#pragma unroll
        for (int j = 0; j < U; ++j) *reinterpret_cast<uint4 *>(stage + stage_off(j * (64 / SEGS) + xtok, xseg)) = xb[j].u;
#pragma unroll
        for (int q = 0; q < U; ++q)
            xo[q] = *reinterpret_cast<const half8_t *>(stage + stage_off(r, PART ? slot * U + q : ((q / OPD) * 4 + slot) * OPD + q % OPD));
    };
    const half_t *cbl = reinterpret_cast<const half_t *>(smem);
    const int set_halves = R * a.E * V;
    auto entry = [&](unsigned idx, int set) {   // entry idx of the concatenated codebooks (LDS) or of the codebook (L2)
        V16 e;
        e.u = make_uint4(0, 0, 0, 0);
        if (L2CB) {
            const unsigned char *p = reinterpret_cast<const unsigned char *>(a.cb) + idx * (unsigned)(V * 2);
            if (V == 8) {
                e = ld16(p);
            } else {
                const V8 t = ld8(p);
                e.w[0] = t.w[0];
                e.w[1] = t.w[1];
            }
        } else {
            const half_t *p = cbl + set + idx * V;
            if (V == 8) {
                e = ld16(p);
            } else {
                const V8 t = ld8(p);
                e.w[0] = t.w[0];
                e.w[1] = t.w[1];
            }
        }
        return e;
    };
    auto load_entries = [&](int it, int u, const V16 (&cd)[RT], V16 (&ev)[U][RT][CPO][R]) {
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int o = u * U + q;
            int set = 0;
            if (!L2CB && a.tiles_k > 1) set = min(op_index(it, o) / a.tile_ops, a.tiles_k - 1) * set_halves;
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int h = 0; h < CPO; ++h)
#pragma unroll
                    for (int rr = 0; rr < R; ++rr)
                        ev[q][t][h][rr] = entry(rr * a.E + skinny_code<CodeT>(cd[t], (o * CPO + h) * R + rr), set);
        }
    };

    // codes of this iteration, of the next one and of the one after that (a wavefront whose iterations have run out
    // repeats the last one and does not use it)
    V16 cd[RT], cn[RT], cf[RT];
    V16 xr[D][U];
    V16 er[L2CB ? 2 : 1][U][RT][CPO][R];
    const int first = min(wave, a.nit - 1);
#pragma unroll
    for (int t = 0; t < RT; ++t) load_codes(first, t, cd[t]);
#pragma unroll
    for (int t = 0; t < RT; ++t) load_codes(min(wave + nwaves, a.nit - 1), t, cn[t]);
#pragma unroll
    for (int e = 0; e < D; ++e) load_x(first, e, xr[e]);
    // scales of the rows that this lane writes at the end, as raw halves (row tile wave % RT; else read there)
    half_t sc4[4];
    {
        const half_t *sp = a.scale ? a.scale : a.x;
#pragma unroll
        for (int i = 0; i < 4; ++i) sc4[i] = sp[a.scale ? min(n0 + 16 * (wave % RT) + 4 * g + i, a.N - 1) : 0];
    }
    if (!L2CB) {
        const half_t *src = a.cb + (a.tile_n > 0 ? (size_t)(n0 / a.tile_n) * a.tiles_k * set_halves : 0);
        const int n16 = set_halves * a.tiles_k / 8;
        for (int i = tid; i < n16; i += blockDim.x) reinterpret_cast<uint4 *>(smem)[i] = reinterpret_cast<const uint4 *>(src)[i];
        __syncthreads();
    }
#pragma unroll
    for (int t = 0; t < RT; ++t) transpose(cd[t]);
    if (L2CB) load_entries(first, 0, cd, er[0]);

    float4v_t acc[RT][CT];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[t][c] = float4v_t{0.f, 0.f, 0.f, 0.f};

    half8_t xo[U];
    {   // element 0 is staged ahead, and so is every next element before the current one is multiplied
        stage_x(xr[0], xo);
        load_x(D < EPI ? first : min(first + nwaves, a.nit - 1), D % EPI, xr[0]);
    }
    for (int it = wave; it < a.nit; it += nwaves) {
        const int nx = min(it + nwaves, a.nit - 1);
        const bool tail = (it + 1) * 4 * MPI > a.ops;   // some lanes of this iteration are past the end of the row
#pragma unroll
        for (int t = 0; t < RT; ++t) load_codes(min(it + 2 * nwaves, a.nit - 1), t, cf[t]);
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            if (L2CB) {
                if (u + 1 == NU) {
#pragma unroll
                    for (int t = 0; t < RT; ++t) {
                        cd[t] = cn[t];
                        transpose(cd[t]);
                    }
                }
                load_entries(u + 1 < NU ? it : nx, (u + 1) % NU, cd, er[(u + 1) & 1]);
            } else {
                load_entries(it, u, cd, er[0]);
            }
            // the operands: one entry, or the fp16 sum of two (one rounding, that of their fp32 sum)
            V16 op[U][RT];
#pragma unroll
            for (int q = 0; q < U; ++q) {
#pragma unroll
                for (int t = 0; t < RT; ++t) {
                    const V16 (&e)[CPO][R] = er[L2CB ? u & 1 : 0][q][t];
#pragma unroll
                    for (int h = 0; h < CPO; ++h) {
#pragma unroll
                        for (int p = 0; p < V / 2; ++p) {
                            half2_t s = e[h][0].h2[p];
                            if (R == 2) s += e[h][R - 1].h2[p];
                            op[q][t].h2[h * (V / 2) + p] = s;
                        }
                    }
                }
            }
            if (tail) {
#pragma unroll
                for (int q = 0; q < U; ++q)
                    if (op_index(it, u * U + q) >= a.ops) {
#pragma unroll
                        for (int t = 0; t < RT; ++t) op[q][t].u = make_uint4(0, 0, 0, 0);
                    }
            }
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const int e = u * CT + c;
                half8_t xc[U];
#pragma unroll
                for (int q = 0; q < U; ++q) xc[q] = xo[q];
                stage_x(xr[(e + 1) % D], xo);
                {
                    const int f = e + 1 + D;   // element f of this iteration, or of one of the next two
                    load_x(f < EPI ? it : f < 2 * EPI ? nx : min(it + 2 * nwaves, a.nit - 1), f % EPI, xr[(e + 1) % D]);
                }
                if (tail) {
#pragma unroll
                    for (int q = 0; q < U; ++q)
                        if (op_index(it, u * U + q) >= a.ops) xc[q] = half8_t{0, 0, 0, 0, 0, 0, 0, 0};
                }
#pragma unroll
                for (int q = 0; q < U; ++q)
#pragma unroll
                    for (int t = 0; t < RT; ++t) acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(op[q][t].h8, xc[q], acc[t][c], 0, 0, 0);
            }
        }
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            if (!L2CB) {
                cd[t] = cn[t];
                transpose(cd[t]);
            }
            cn[t] = cf[t];
        }
    }

    // partial tiles -> LDS [tile][wavefront][lane] (over the codebooks), added in wavefront order, tile t by wavefront t
    // mod the wavefronts.  Lane (r, g) of a tile holds token r, rows 4 g + 0..3.
    float4v_t *red = reinterpret_cast<float4v_t *>(smem);
    __syncthreads();
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int t = 0; t < RT; ++t) red[((c * RT + t) * nwaves + wave) * 64 + lane] = acc[t][c];
    __syncthreads();
    for (int i = wave; i < RT * CT; i += nwaves) {
        float4v_t sum = red[(i * nwaves) * 64 + lane];
        for (int w = 1; w < nwaves; ++w) sum += red[(i * nwaves + w) * 64 + lane];
        const int t = i % RT, m = m0 + 16 * (i / RT) + r, n = n0 + 16 * t + 4 * g;
        if (m >= a.M) continue;
        half4_t o;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float sc = !a.scale ? 1.f : t == wave % RT ? (float)sc4[j] : (float)a.scale[min(n + j, a.N - 1)];
            o[j] = (half_t)(sum[j] * sc);
        }
        half_t *yp = a.y + (size_t)m * a.N + n;
        if ((a.N & 3) == 0) {
            if (n < a.N) *reinterpret_cast<half4_t *>(yp) = o;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (n + j < a.N) yp[j] = o[j];
        }
    }
}

// Elements of X of one launch: its kernel holds byte offsets into X in 32 bits.  At least 384 tokens (K <= 2^22), whole
// tiles of every kind.
constexpr long kSkinnyMaxX = 1L << 31;
int skinny_max_tokens(int K) { return (int)std::min(1L << 30, (kSkinnyMaxX - 1) / K / 128 * 128); }

constexpr size_t kSkinnyLds = 160 * 1024, kSkinnyLdsCodebook = 128 * 1024;
template <typename CodeT, int V, int R>
constexpr int skinny_unit_of() {
    constexpr int BITS = SkinnyShape<CodeT, V, R>::BITS, LB = SkinnyShape<CodeT, V, R>::LB, CPO = 8 / V;
    constexpr int MPI = LB * 8 / (BITS * R * CPO);
    return skinny_unit(MPI, LB != 12 && BITS * R * CPO <= 32 ? MPI / (LB / 4) : MPI);
}

template <typename CodeT, int V, int R, bool L2CB, int RT, int CT>
int run_tile(const vq_weight_t *w, const half_t *x, int M, half_t *y, hipStream_t s) {
    constexpr int MPI = SkinnyShape<CodeT, V, R>::LB * 8 / (SkinnyShape<CodeT, V, R>::BITS * R * (8 / V));
    SkinnyArgs a;
    a.codes = w->codes;
    a.cb = (const half_t *)w->codebooks;
    a.scale = (const half_t *)w->scale;
    a.x = x;
    a.y = y;
    a.N = w->N;
    a.K = w->K;
    a.M = M;
    a.E = w->n_entries;
    a.ops = w->K / 8;
    a.nit = (a.ops + 4 * MPI - 1) / (4 * MPI);
    a.tile_n = w->cb_tile_n;
    a.tiles_k = w->cb_tile_n > 0 ? w->K / w->cb_tile_k : 1;
    a.tile_ops = w->cb_tile_n > 0 ? w->cb_tile_k / 8 : 1;
    a.groups_m = (M + 16 * CT - 1) / (16 * CT);
    constexpr size_t kUnit = 1024 * skinny_unit_of<CodeT, V, R>();
    const size_t cb_bytes = L2CB ? 0 : ((size_t)R * a.E * V * 2 * a.tiles_k + 15) & ~(size_t)15;
    const long grid = (long)((w->N + 16 * RT - 1) / (16 * RT)) * a.groups_m;
    constexpr int kMaxWaves = skinny_max_waves(L2CB, RT, CT);
    auto lds_of = [&](int n) { return std::max(cb_bytes + n * kUnit, (size_t)RT * CT * n * 1024); };
    // a wavefront per iteration over K
    int waves = std::min(a.nit, kMaxWaves);
    while (waves > 1 && cb_bytes + waves * kUnit > kSkinnyLds) waves = (waves + 1) / 2;
    // and more where a short K leaves few of them to stage the codebooks (one wavefront: 20 us for 128 KiB), unless that takes
    // the place of other workgroups
    auto per_cu = [&](int n) { return std::min((int)(kSkinnyLds / lds_of(n)), kMaxWaves / n); };
    for (int n = std::min((int)(cb_bytes / 8192), kMaxWaves); n > waves; --n)
        if (lds_of(n) <= kSkinnyLds && (grid <= 256 || per_cu(n) == per_cu(waves))) waves = n;
    const size_t lds = lds_of(waves);
    static KernelSetup setup;
    if (int st = kernel_setup(reinterpret_cast<const void *>(&gemm_skinny_kernel<CodeT, V, R, L2CB, RT, CT>), lds, false, setup)) return st;
    gemm_skinny_kernel<CodeT, V, R, L2CB, RT, CT><<<(int)grid, waves * 64, lds, s>>>(a);
    return launch_status();
}

// The tiles that are built, {RT, CT}.
struct SkinnyTile { int rt, ct; };
constexpr SkinnyTile kLdsTiles[] = {{1, 1}, {1, 2}, {2, 2}, {2, 4}, {4, 4}};   // ({1, 4} was never the best)
constexpr SkinnyTile kL2Tiles[] = {{1, 1}, {1, 2}, {1, 4}, {2, 4}, {1, 8}, {2, 8}};

// Estimated clocks of a launch: a workgroup's lookups (3.5 per clock from LDS, 0.35 from L2) and X (41 bytes per clock)
// plus its start and end, times the rounds of workgroups over 256 CUs.  From LDS a second round is a whole one, later
// ones fill in; from L2 all workgroups share the dies' L2s, so fewer than 256 of them are not that much faster.
// The constants were fitted to 210 measured shapes (six formats, N 256 .. 11008, M 17 .. 256) x 6 tiles: the tile that
// this picks takes 0.5 % more than the best one on average and 17 % more at worst.  Staging of the codebooks, the same for every
// tile, counts only in the estimate (*clocks).
int skinny_tile(const vq_weight_t *w, int M, bool l2, double staging = 0, double *us = nullptr) {
    int best = 0;
    double best_cost = 1e300;
    for (int i = 0; i < (l2 ? 6 : 5); ++i) {
        const SkinnyTile t = l2 ? kL2Tiles[i] : kLdsTiles[i];
        if (w->cb_tile_n > 0 && w->cb_tile_n % (16 * t.rt) != 0) continue;
        if (w->code_bits == 12 && t.rt == 4) continue;   // (four operands per lane and unit: does not fit the registers)
        const double r = (double)(((long)w->N + 16 * t.rt - 1) / (16 * t.rt)) * ((M + 16 * t.ct - 1) / (16 * t.ct)) / 256;
        const double rounds = l2 ? (r <= 1 ? std::max(0.7, r) : r + 0.3) : r <= 1 ? 1.0 : r <= 2 ? 2.0 : r + 0.3;
        const double lookups = 16.0 * t.rt * (w->K / w->v) * w->n_codebooks / (l2 ? 0.35 : 3.5);
        const double cost = rounds * (lookups + 16.0 * t.ct * w->K * 2 / 41 + 2000 + staging);
        if (cost < best_cost) {
            best_cost = cost;
            best = i;
            // (to compare with another kernel: fitted to 397 measured launches, 11 % off on average)
            const double x = 16.0 * t.ct * w->K * 2 / 41;
            if (us && l2) *us = rounds * (lookups * (w->v == 8 ? 2.88e-4 : 3.34e-4) + x * 5.7e-4 + 1.26) + 2.7;
            if (us && !l2) *us = rounds * (lookups * (w->v == 8 ? 2.81e-4 : 1.83e-4) + x * 6.6e-4 + staging * 6.3e-4 + 2.26) + 1.4;
        }
    }
    return best;
}

template <typename CodeT, int V, int R>
int run_lds(int tile, const vq_weight_t *w, const half_t *x, int M, half_t *y, hipStream_t s) {
    switch (tile) {
        case 0: return run_tile<CodeT, V, R, false, 1, 1>(w, x, M, y, s);
        case 1: return run_tile<CodeT, V, R, false, 1, 2>(w, x, M, y, s);
        case 2: return run_tile<CodeT, V, R, false, 2, 2>(w, x, M, y, s);
        case 3: return run_tile<CodeT, V, R, false, 2, 4>(w, x, M, y, s);
        default:
            if constexpr (!std::is_same<CodeT, Code12>::value) return run_tile<CodeT, V, R, false, 4, 4>(w, x, M, y, s);
            return VQ_ERR_UNSUPPORTED;
    }
}
template <int V>
int run_l2(int tile, const vq_weight_t *w, const half_t *x, int M, half_t *y, hipStream_t s) {
    switch (tile) {
        case 0: return run_tile<uint16_t, V, 1, true, 1, 1>(w, x, M, y, s);
        case 1: return run_tile<uint16_t, V, 1, true, 1, 2>(w, x, M, y, s);
        case 2: return run_tile<uint16_t, V, 1, true, 1, 4>(w, x, M, y, s);
        case 3: return run_tile<uint16_t, V, 1, true, 2, 4>(w, x, M, y, s);
        case 4: return run_tile<uint16_t, V, 1, true, 1, 8>(w, x, M, y, s);
        default: return run_tile<uint16_t, V, 1, true, 2, 8>(w, x, M, y, s);
    }
}

bool codebooks_fit_lds(const vq_weight_t *w) {
    const size_t sets = w->cb_tile_n > 0 ? w->K / w->cb_tile_k : 1;
    return sets * w->n_codebooks * w->n_entries * w->v * 2 <= kSkinnyLdsCodebook;
}
// Entries from LDS: the codebooks fit, and their sets are whole 16-byte pieces (an odd number of 8-byte entries is not;
// one uint16 codebook of those is looked up in L2 like a large one).
bool entries_from_lds(const vq_weight_t *w) {
    return codebooks_fit_lds(w) && (w->n_codebooks * w->n_entries * w->v * 2) % 16 == 0;
}

int run_skinny(int tile, const vq_weight_t *w, const half_t *x, int M, half_t *y, hipStream_t s) {
    if (!entries_from_lds(w)) return w->v == 8 ? run_l2<8>(tile, w, x, M, y, s) : run_l2<4>(tile, w, x, M, y, s);
#define VQ_SK(CodeT)                                                                                              \
    if (w->v == 8) return w->n_codebooks == 1 ? run_lds<CodeT, 8, 1>(tile, w, x, M, y, s) : run_lds<CodeT, 8, 2>(tile, w, x, M, y, s); \
    return w->n_codebooks == 1 ? run_lds<CodeT, 4, 1>(tile, w, x, M, y, s) : run_lds<CodeT, 4, 2>(tile, w, x, M, y, s);
    if (w->code_bits == 8) { VQ_SK(uint8_t) }
    if (w->code_bits == 12) { VQ_SK(Code12) }
    VQ_SK(uint16_t)
#undef VQ_SK
}

}  // namespace

// One or two codebooks, whole code loads per row (16-byte aligned rows; 8 bytes for single uint8 codes, 12-byte words
// for 12-bit codes), codebooks that can be staged in LDS -- or one uint16 codebook of any size, from L2.
bool gemm_skinny_supported(const vq_weight_t *w) {
    const int R = w->n_codebooks;
    if (R != 1 && R != 2) return false;
    const int lb = w->code_bits == 12 ? 12 : R * w->code_bits == 8 ? 8 : 16;
    const long row_bits = (long)(w->K / w->v) * R * w->code_bits;
    if (w->K <= 0 || w->K % 8 != 0 || w->N <= 0 || w->N > (1 << 26) || row_bits % (lb * 8) != 0 || w->K > (1 << 22)) return false;   // (256 tokens: byte offsets into X of 32 bits)
    return entries_from_lds(w) || (w->cb_tile_n == 0 && R == 1 && w->code_bits == 16);
}

// More than 256 tokens: against the two-stage product, which writes the weight once and multiplies it tile by tile.  Measured,
// two-stage / here, us: two 256-entry codebooks, N = 256, K = 4096, 1024 tokens 18.7 / 9.1; N = 1024, K = 2048, 400 tokens 12.0 / 9.0,
// 2048 tokens 18.0 / 21.2; N = K = 4096, 400 tokens 33.6 / 31.4, 700 tokens 41.5 / 48.5; N = 11008, K = 1024, 257 tokens 28.7 / 24.0; 2^16
// entries, N = 64, K = 8192, 257 tokens 25.2 / 13.2.  Every workgroup stages the codebooks (41 bytes per clock).  The estimates are
// good to about 10 %: over 397 measured calls (8 formats, 11 weights, 257 to 2048 tokens) the pick takes 1.9 % more than the
// better of the two on average.  (A supported weight with K % 64 == 0.)
bool gemm_skinny_wins(const vq_weight_t *w, int M) {
    if ((long)M * w->K >= kSkinnyMaxX) return false;
    double here;
    const bool l2 = !entries_from_lds(w);
    const size_t sets = w->cb_tile_n > 0 ? w->K / w->cb_tile_k : 1;
    skinny_tile(w, M, l2, l2 ? 0 : sets * w->n_codebooks * w->n_entries * w->v * 2 / 41.0, &here);
    // dequantization: by the million elements, the first 16 of which are dearer (few wavefronts), and launches
    const double m = 1e-6 * w->N * w->K, first = std::min(m, 16.0), rest = m - first;
    const double two = 3.5 + 0.97 * gemm_tiles_time(M, w->N, w->K, nullptr) +
                       (l2 ? w->v == 8 ? 1.33 * first + 0.62 * rest : 1.76 * first + 1.09 * rest : w->v == 8 ? 1.29 * first + 0.45 * rest : 1.26 * first + 0.57 * rest);
    return (l2 ? 0.92 : 1.0) * here < two;
}

// Where vq_gemv (1 .. 16 tokens) runs here.
// A codebook that does not fit LDS: the row kernel gathers every entry once per 4 tokens (and per token beyond 256 code
// chunks a row), this one once.  v = 8 from two tokens on (N = K = 4096: 13.1 / 11.7 us; 16 tokens 67.4 / 12.4; one token
// 12.0 / 11.8 at 4096 rows but 26.9 / 28.9 at 11008), v = 4 from five on (4 tokens 21.0 / 20.4, at 11008 rows 48.0 / 53.3;
// 8 tokens 41.2 / 20.6).  Not where the caller says that the front of the codebook is hot: that part is kept in LDS.
// LDS codebooks: the matrix-core gemv reads X in operand order, which costs it 0.1 .. 0.4 us per token; from 14 tokens on
// this kernel is ahead where one round of workgroups covers the rows (16 tokens, N = 4096, K = 11008, two codebooks
// 13.6 / 11.2; 8 tokens 10.3 / 10.9; 16 tokens of 11008 rows 15.0 / 18.4) and K is long enough to fill its wavefronts.  Its
// time over the other's with 14 .. 16 tokens, N = 256 .. 4096: v = 8, K = 1024 1.00 .. 1.04, 2048 0.93 .. 1.03, 4096 0.83 .. 1.01; v = 4
// with uint16 codes, K = 1024 1.04 .. 1.07, 2048 0.96 .. 1.01; with uint8 codes, one codebook, 2048 1.01 .. 1.06, 4096 0.84 .. 0.90, two,
// 2048 1.02 .. 1.07, 4096 0.98 .. 1.04, 6400 0.87 .. 0.94.  Not for 12-bit codes, which have no transposition (16 tokens with cold
// caches, N = K = 4096: 10.1 / 10.7).
bool gemm_skinny_for_gemv(const vq_weight_t *w, int bs) {
    if (!gemm_skinny_supported(w)) return false;
    if (codebooks_fit_lds(w)) {
        const int long_k = w->v == 8 || w->code_bits == 16 ? 2048 : w->n_codebooks == 1 ? 4096 : 5120;
        return entries_from_lds(w) && bs >= 14 && w->code_bits != 12 && w->K >= long_k && w->N <= 16 * 256;
    }
    if (gemv_mfma_supported(w)) return false;
    return bs >= (w->v == 8 ? 2 : 5) || w->K / (8 * w->v) > 256;
}

int launch_gemm_skinny(const vq_weight_t *w, const void *x, int M, void *y, hipStream_t s) {
    const half_t *xp = (const half_t *)x;
    half_t *yp = (half_t *)y;
    const int most = skinny_max_tokens(w->K);   // of a launch; the rest in further ones
    for (int m = 0; m < M; m += most) {
        const int n = std::min(most, M - m);
        if (int st = run_skinny(skinny_tile(w, n, !entries_from_lds(w)), w, xp + (size_t)m * w->K, n, yp + (size_t)m * w->N, s)) return st;
    }
    return VQ_OK;
}

}  // namespace vq
