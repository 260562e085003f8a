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
#include <cmath>
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
#include "gemm_skinny_body.inc"
}
// 48 tokens: what X costs a workgroup is by the token, and one of 33 to 48, or two of 65 to 96, read a quarter less than with 64.
// 4096 x 4096, two 256-entry codebooks, 77 tokens 12.8 -> 11.3 us, 48 tokens 10.4 -> 9.2; one, K = 11008, 80 tokens 23.1 -> 18.3.
template <typename CodeT, int V, int R, int RT>
__global__ __launch_bounds__(64 * skinny_max_waves(false, RT, 3)) void gemm_skinny_48_kernel(SkinnyArgs a) {
    constexpr bool L2CB = false;
    constexpr int CT = 3;
#include "gemm_skinny_body.inc"
}

// Elements of X of one launch: its kernel holds byte offsets into X in 32 bits.  At least 384 tokens (K <= 2^22), whole tiles of
// every kind that launches of more than 256 tokens have (not the 48 tokens).
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
    void (*kernel)(SkinnyArgs);
    if constexpr (CT == 3)
        kernel = &gemm_skinny_48_kernel<CodeT, V, R, RT>;
    else
        kernel = &gemm_skinny_kernel<CodeT, V, R, L2CB, RT, CT>;
    if (int st = kernel_setup(reinterpret_cast<const void *>(kernel), lds, false, setup)) return st;
    kernel<<<(int)grid, waves * 64, lds, s>>>(a);
    return launch_status();
}

// The tiles that are built, {RT, CT}.
struct SkinnyTile { int rt, ct; };
constexpr SkinnyTile kLdsTiles[] = {{1, 1}, {1, 2}, {2, 2}, {2, 4}, {4, 4}, {2, 3}, {1, 3}};   // ({1, 4} was never the best)
constexpr SkinnyTile kL2Tiles[] = {{1, 1}, {1, 2}, {1, 4}, {2, 4}, {1, 8}, {2, 8}};

// Estimated clocks of a launch: a workgroup's lookups (3.5 per clock from LDS, 0.35 from L2) and X (41 bytes per clock)
// plus its start and end, times the rounds of workgroups over 256 CUs.  From LDS a second round is a whole one, later
// ones fill in; from L2 all workgroups share the dies' L2s, so fewer than 256 of them are not that much faster.
// The constants were fitted to 210 measured shapes (six formats, N 256 .. 11008, M 17 .. 256) x 6 tiles; over 1950 others (15
// formats, N 16 .. 11008, K 256 .. 11008) the tile that this picks takes 2.7 % more than the best one on average and 43 % or more in the
// worst hundredth, mostly below K = 512 (8.9 %), where a workgroup has fewer wavefronts than its tile could feed; K > 2048 1.1 %.  Staging
// of the codebooks, the same for every tile, counts only in the estimate (*us).
int skinny_tile(const vq_weight_t *w, int M, bool l2, double staging = 0, double *us = nullptr) {
    int best = 0;
    double best_cost = 1e300;
    for (int i = 0; i < (l2 ? 6 : 7); ++i) {
        const SkinnyTile t = l2 ? kL2Tiles[i] : kLdsTiles[i];
        if (w->cb_tile_n > 0 && w->cb_tile_n % (16 * t.rt) != 0) continue;
        if (t.ct == 3 && M > 256) continue;   // (X no longer fits a die's L2, and more workgroups that read it lose: N = 256, K = 4096, 700 tokens 10.1 -> 11.7)
        if (w->code_bits == 12 && t.rt == 4) continue;   // (four operands per lane and unit: does not fit the registers)
        const double r = (double)(((long)w->N + 16 * t.rt - 1) / (16 * t.rt)) * ((M + 16 * t.ct - 1) / (16 * t.ct)) / 256;
        const double rounds = l2 ? (r <= 1 ? std::max(0.7, r) : r + 0.3) : r <= 1 ? 1.0 : r <= 2 ? 2.0 : r + 0.3;
        const double lookups = 16.0 * t.rt * (w->K / w->v) * w->n_codebooks / (l2 ? 0.35 : 3.5);
        // (16 rows x 48 tokens of one codebook of v = 4, whose lookups are few, read too much of X where K is long: 4096 x 11008, 46 tokens 15.8 -> 16.5,
        // 585 x 10688, 219 tokens 15.4 -> 16.7)
        if (t.ct == 3 && t.rt == 1 && w->v == 4 && w->n_codebooks == 1 && w->K > 8192) continue;
        const double cost = rounds * (lookups + 16.0 * t.ct * w->K * 2 / 41 + 2000 + staging);
        if (cost < best_cost) {
            best_cost = cost;
            best = i;
            // (to compare with another kernel: constants by the formats' entries, and the start and end of a workgroup by its tile)
            const double x = 16.0 * t.ct * w->K * 2 / 41, ends = t.rt * t.ct * (r <= 1 ? 0.1 : r <= 2 ? 0.24 : 0.25 * (0.7 * std::ceil(r) + 0.3 * r));
            if (us && l2) *us = rounds * (lookups * (w->v == 8 ? 2.88e-4 : 3.34e-4) + x * 5.7e-4 + 1.26) + ends + 2.7;
            if (us && !l2) *us = rounds * (lookups * (w->v == 8 ? 2.81e-4 : 1.83e-4) + x * 6.6e-4 + staging * 6.3e-4 + 2.26) + ends + 1.4;
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
        case 5: return run_tile<CodeT, V, R, false, 2, 3>(w, x, M, y, s);
        case 6: return run_tile<CodeT, V, R, false, 1, 3>(w, x, M, y, s);
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

// The tile of a launch of M tokens, 16 {weight rows} + {tokens} in sixteens (for tests).
int gemm_skinny_tile_of(const vq_weight_t *w, int M) {
    const bool l2 = !entries_from_lds(w);
    const SkinnyTile t = (l2 ? kL2Tiles : kLdsTiles)[skinny_tile(w, M, l2)];
    return 16 * t.rt + t.ct;
}

// More than 256 tokens: against the two-stage product, which writes the weight once and multiplies it tile by tile.  Measured,
// two-stage / here, us: two 256-entry codebooks, N = 256, K = 4096, 1024 tokens 18.7 / 9.1; N = 1024, K = 2048, 400 tokens 12.0 / 9.0,
// 2048 tokens 18.0 / 21.2; N = K = 4096, 400 tokens 33.6 / 31.4, 700 tokens 41.5 / 48.5; N = 11008, K = 2112, 327 tokens 38.5 / 63.5; two
// of 4096 entries, N = 11008, K = 10560, 317 tokens 230 / 149; 2^16 entries, N = 64, K = 8192, 257 tokens 25.2 / 13.2.  Every workgroup
// stages the codebooks (41 bytes per clock).  What the estimates have to know: here, that a workgroup of a large tile takes longer to start
// and to end, and that rounds are mostly whole ones; of the two stages, that the output is written (element by element where N % 8 != 0),
// that lookups are dearer the less of the codebooks a CU's L1 holds, and that a weight of more than 64 M elements does not stay in the
// Infinity Cache.  Over 8372 measured calls (15 formats, N 16 .. 11008, K 256 .. 11008, 257 to 4096 tokens) the pick takes 0.7 % more
// than the better of the two on average, 23 % or more in the worst hundredth.  (A supported weight with K % 64 == 0.)
bool gemm_skinny_wins(const vq_weight_t *w, int M) {
    if ((long)M * w->K >= kSkinnyMaxX) return false;
    double here;
    const bool l2 = !entries_from_lds(w);
    const size_t sets = w->cb_tile_n > 0 ? w->K / w->cb_tile_k : 1, set = (size_t)w->n_codebooks * w->n_entries * w->v * 2;
    skinny_tile(w, M, l2, l2 ? 0 : sets * set / 41.0, &here);
    // in millions: the weight's elements (the first 16 of which are dearer: few wavefronts), lookups, outputs
    const double m = 1e-6 * w->N * w->K, first = std::min(m, 16.0), rest = m - first, far = std::max(m - 64, 0.0);
    const double lookup = m / w->v * w->n_codebooks, out = 1e-6 * w->N * M;
    const double two = 4.0 + 1.05 * gemm_tiles_time(M, w->N, w->K, nullptr) + 0.76 * first + 0.14 * rest + 0.79 * far +
                       lookup * (set > 128 * 1024 ? 2.92 : set > 32 * 1024 ? 1.63 : 0.71) + out * (w->N % 8 != 0 ? 1.96 : 0.3);
    return here < two;
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
