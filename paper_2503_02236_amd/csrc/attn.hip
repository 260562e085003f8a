// VQ-attn (decode) for gfx950: out[b][h] = softmax_t(sm_scale * q . K[t]) . V[t] over a KV
// cache stored as uint8 VQ codes.  Formula: VQ-LLM (arXiv 2503.02236) Sec. II-B; setup
// VQ<4,8,1>, 32 heads x 128 channels: Sec. III-A; token-parallel split with a merge of the
// local softmax statistics: Sec. III-B (flash-decoding dataflow of Fig. 5).
//
// Mapping (wave64): four lanes share a token.  Lane (tok = lane % 16, g = lane / 16) owns channels
// [32 g, 32 g + 32) of token tok of the current 16-token step.
//   K side: the scores come from the matrix cores.  v_mfma_f32_16x16x32_f16 takes, per lane, 8
//   consecutive k of one column as its B operand: with k = channel and column = token that is
//   8 / v dequantized sub-vectors of the lane's token, gathered from the LDS codebook straight into the
//   operand registers (layout fusion, Sec. VI-B: no shuffle, no LDS round trip).  The A operand is q,
//   the same in all 16 rows, so every accumulator row holds the score and each of a token's four
//   lanes reads its token's score from its own registers.  Four MFMAs cover the 128 channels.
//   V side: the lane dequantizes its 32 channels of the token's V vector and adds p_t * V[t] into 32
//   PRIVATE fp32 accumulators.  The column-wise accumulation over tokens that forces a shared-memory
//   round trip in the paper's baseline (Sec. III-B, Fig. 6) is deferred to one butterfly over the 16
//   token lanes at the very end, so dequantized values never travel through LDS.
// p V on the matrix cores (entries through the transposing LDS read, weights as two halves) halves the vector instructions
// and was not faster: its chain per tile is longer.  B = 16, H = 32, T = 4096, one codebook per head and side 30.1 us here, 31.9
// there (codes in the last-level cache); 32 codebooks 34.9 / 37.6; 0 to 9 % in favour of this over 140 shapes.
// Only ~130 registers per lane are needed, so 16 wavefronts per CU hide the gather latency.
// Codebooks live in LDS (2 KB each for one codebook per head and side).
//
// A workgroup streams over its token range in tiles of 16 code bytes per lane and side (32 tokens
// per wavefront for v = 4).  The codes of the
// next two tiles are in flight while a tile is processed (register double buffers), so the HBM stream
// and the LDS gathers overlap.  Softmax is kept online per wavefront: a wave-uniform running
// maximum; the accumulators are rescaled only when a tile raises it (rare after the first tiles).
#include <cfloat>

#include "vq_common.h"

namespace vq {

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kAttnMinTokens = 512;   // do not split token ranges below this
constexpr int kAttnTargetWgs = 512;   // two workgroups per compute unit

constexpr int kAttnWaves = 8;   // wavefronts per workgroup
// 16-token steps per wavefront and tile: 16 bytes of codes per lane, tile and side
constexpr int attn_steps(int v) { return v / 2; }
constexpr int attn_tile(int v) { return kAttnWaves * 16 * attn_steps(v); }  // tokens per workgroup and tile

struct AttnArgs {
    const uint8_t *k_codes, *v_codes;
    const half_t *k_cb, *v_cb;
    const int *seq_lens;
    const half_t *q;
    half_t *out;
    float *ws;      // [B*H][S][D + 2] partials when S > 1
    int B, H, T, E, G, S;
    int tc;         // tokens per workgroup (token-range split), a multiple of the tile
    int pg_shift;   // log2 of sub-vectors per codebook group
    float scale2;   // sm_scale * log2(e)
};

// Butterfly sum of acc[0..32) over the 16 lanes of a row (lanes that share lane / 16); afterwards
// lane l holds the totals of elements 2 (l % 16) and 2 (l % 16) + 1 in acc[0], acc[1].  In every step
// a lane keeps one half of its values and adds the partner lane's copy of that half.
__device__ __forceinline__ void row_reduce_scatter(float (&acc)[32], int lane) {
#pragma unroll
    for (int step = 0; step < 4; ++step) {
        const int m = 8 >> step;        // lane mask
        const int half = 16 >> step;    // elements kept
        const bool upper = (lane & m) != 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            if (i < half) {
                float lo = acc[i], hi = acc[i + half];
                float send = upper ? lo : hi;
                float keep = upper ? hi : lo;
                acc[i] = keep + __shfl_xor(send, m, 64);
            }
        }
    }
}

// Maximum over the wavefront as a wave-uniform value, on the vector ALU only (lane permutes inside
// rows of 16, then one read per row), so it does not queue behind the LDS gathers.
template <int CTRL>
__device__ __forceinline__ float dpp_max_step(float x) {
    int y = __builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(x), CTRL, 0xF, 0xF, false);
    return fmaxf(x, __int_as_float(y));
}
__device__ __forceinline__ float wave_max_uniform(float x) {
    x = dpp_max_step<0xB1>(x);   // quad_perm [1,0,3,2]
    x = dpp_max_step<0x4E>(x);   // quad_perm [2,3,0,1]
    x = dpp_max_step<0x141>(x);  // row_half_mirror
    x = dpp_max_step<0x140>(x);  // row_mirror: every lane now holds the maximum of its row of 16
    const int xi = __float_as_int(x);
    const float r0 = __int_as_float(__builtin_amdgcn_readlane(xi, 0));
    const float r1 = __int_as_float(__builtin_amdgcn_readlane(xi, 16));
    const float r2 = __int_as_float(__builtin_amdgcn_readlane(xi, 32));
    const float r3 = __int_as_float(__builtin_amdgcn_readlane(xi, 48));
    return fmaxf(fmaxf(r0, r1), fmaxf(r2, r3));
}

// Load of one codebook entry (v halves) from an LDS byte address into bytes [at, at + 2 v) of a
// 64-byte register block.
template <int V>
__device__ __forceinline__ void lds_entry_into(V16 (&blk)[4], int at, unsigned addr) {
    if constexpr (V == 8) {
        typedef unsigned raw_t __attribute__((ext_vector_type(4)));
        const raw_t r = *reinterpret_cast<const __attribute__((address_space(3))) raw_t *>((uintptr_t)addr);
        blk[at / 16].w[0] = r.x; blk[at / 16].w[1] = r.y; blk[at / 16].w[2] = r.z; blk[at / 16].w[3] = r.w;
    } else if constexpr (V == 4) {
        typedef unsigned raw_t __attribute__((ext_vector_type(2)));
        const raw_t r = *reinterpret_cast<const __attribute__((address_space(3))) raw_t *>((uintptr_t)addr);
        blk[at / 16].w[(at % 16) / 4] = r.x; blk[at / 16].w[(at % 16) / 4 + 1] = r.y;
    } else {
        blk[at / 16].w[(at % 16) / 4] = *reinterpret_cast<const __attribute__((address_space(3))) unsigned *>((uintptr_t)addr);
    }
}

// (byte B of w) << sh.  With the shift out of the compiler's sight this is one instruction (a shift that selects the
// byte); with a constant it is an extract and a shift.  (Not written as assembly: the compiler keeps its own vector
// instructions clear of registers that a matrix instruction has yet to write, but not those of an asm statement.)
template <int B>
__device__ __forceinline__ unsigned byte_shl(unsigned w, unsigned sh) {
    return ((w >> (8 * B)) & 0xFFu) << (sh & 31u);
}

// ONE: a single codebook per head and side (cb_groups == 1, at most 4 KiB each): the K codebook
// sits at LDS offset 0 and the V codebook at 4096, so an entry's address is (code * v * 2) plus a
// constant that folds into the offset field of the LDS instruction.
//
// The lookups of a tile form one sequence of groups (per 16-token step: the lane's 32 K channels, later
// its 32 V channels); the LDS gathers of group n+1 are written before the arithmetic of group n, and the
// sequence continues across the K/V boundary and into the next tile, so the LDS queue never drains.
//
// SEQ: items (token ranges of batch entries) per workgroup (1 or 2).  With 2, wavefronts 0-7 and 8-15 attend
// two items of the SAME head and share its codebooks in LDS: the layout with one codebook per sub-space needs
// 128 KiB for them, so only one workgroup fits a CU, and this keeps 16 wavefronts on it and stages the
// codebooks once per pair.
//
// REP (v = 4, one codebook per head and side): every entry is stored 32 times, copy c of entry e at byte
// e * 256 + c * 8, and lane l reads copy l % 32.  LDS serves the 8-byte reads of 32 consecutive lanes in one pass
// if they fall into 32 different 8-byte columns (address / 8 mod 32) and needs one more pass per further address
// in a column: the 32 lanes of a pass now sit in 32 different columns whatever their codes are, where random
// entries of one shared copy take 2.4 passes (the paper's takeaway on shared-memory bank conflicts, Sec. III-B).
// 64 KiB per side; one workgroup of two sequences (SEQ = 2) per compute unit.  An address is one byte
// permute: (code << 8) | lane constant, the V side's constant carrying its base of 64 KiB.
constexpr int kAttnRepCopies = 32;
constexpr int kAttnRepSide = 65536;   // bytes per side: 256 entries x 32 copies x 8 bytes

template <int V, bool ONE, int SEQ, bool REP = false>
__global__ __launch_bounds__(kAttnWaves * 64 * SEQ) __attribute__((amdgpu_waves_per_eu(4, 4))) void attn_decode_kernel(AttnArgs a) {
    static_assert(!REP || (V == 4 && ONE), "replicated codebooks: one codebook of 8-byte entries per side");
    constexpr int D = 128;
    constexpr int P = D / V;          // codes (bytes) per token and side
    constexpr int CB = 32 / V;        // codes (bytes) per lane, step and side: the lane's 32 channels
    constexpr int CW = (CB + 3) / 4;  // dwords holding them
    constexpr int NS = attn_steps(V);
    constexpr int TILE = attn_tile(V);
    constexpr unsigned SH = V == 8 ? 4 : V == 4 ? 3 : 2;  // log2 of the entry size in bytes
    extern __shared__ __align__(16) unsigned char smem[];
    // Entry addresses are formed as plain LDS byte offsets (shifted code + constant), which is only
    // right if the dynamic LDS block starts at LDS address 0: true for a kernel without static LDS.
    // The launcher checks that (kernel_setup) and returns an error instead of launching otherwise.
    const int cb_bytes = a.G * a.E * V * 2;        // per side
    const int v_off = REP ? kAttnRepSide : ONE ? 4096 : cb_bytes;       // LDS offset of the V codebook
    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);   // (a scalar: so are the bases of the code loads)
    const int seq = wid / kAttnWaves, wave = wid % kAttnWaves;  // sequence of the workgroup, wavefront in it
    const int tok = lane & 15, g = lane >> 4;
    // item of this wavefront: a batch entry's token range (pairs: two items in a row)
    const int h = blockIdx.x % a.H, item = SEQ == 1 ? 0 : (blockIdx.x / a.H) * SEQ + seq;
    const int b = SEQ == 1 ? blockIdx.x / a.H : item / a.S, split = SEQ == 1 ? blockIdx.y : item % a.S;
    const bool valid = b < a.B;                      // an odd number of items leaves the last pair half empty
    const int bh = (valid ? b : 0) * a.H + h;
    float *norms = reinterpret_cast<float *>(smem + 2 * (size_t)v_off);   // REP: [16] largest |entry|^2 of K, a share of the entries each
    float *xw = norms + (REP ? 16 : 0) + seq * (kAttnWaves * (D + 2));  // [waves][D] + [waves] + [waves]
    float *xw_m = xw + kAttnWaves * D, *xw_l = xw_m + kAttnWaves;
    const int len = !valid ? 0 : a.seq_lens ? min(max(a.seq_lens[b], 0), a.T) : a.T;
    const int start = split * a.tc;
    const int end = min(len, start + a.tc);  // this sequence attends tokens [start, end) here
    // nothing to attend in this token range: the wavefronts still take part in the barriers and
    // deliver an empty partial result (uniform over the wavefronts of a sequence)
    const bool active = start < end;

    const int ntiles = active ? (end - start + TILE - 1) / TILE : 0;
    const size_t row0 = (size_t)bh * a.T;
    // token of (tile it, step s) for this lane, counted from the start of the range: t_lane + it * TILE + s * 16
    const int t_lane = wave * (16 * NS) + tok, count = end - start;

    // codes of one tile and side -> registers (the lane's CB bytes of each of its NS tokens); tokens
    // past the end re-read the last valid token (their scores are masked)
    // (byte offsets of 32 bits: a range that did not fit them would be part of a cache of hundreds of gigabytes)
    const uint8_t *k_base = a.k_codes + (row0 + start) * P, *v_base = a.v_codes + (row0 + start) * P;
    auto load_codes = [&](const uint8_t *codes, int it, uint32_t (&buf)[NS][CW]) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const uint8_t *cp = codes + (uint32_t)min(t_lane + it * TILE + s * 16, count - 1) * (uint32_t)P + (uint32_t)(g * CB);
            if constexpr (CB == 4) {
                buf[s][0] = *reinterpret_cast<const uint32_t *>(cp);
            } else if constexpr (CB == 8) {
                V8 c = ld8(cp);
                buf[s][0] = c.w[0]; buf[s][1] = c.w[1];
            } else {
                V16 c = ld16(cp);
#pragma unroll
                for (int i = 0; i < 4; ++i) buf[s][i] = c.w[i];
            }
        }
    };

    // 1. codebooks of this head (both sides): global loads first, they are the first to be needed
    const int n16 = cb_bytes / 16;
    const uint4 *ks = reinterpret_cast<const uint4 *>(a.k_cb + (size_t)h * (cb_bytes / 2));
    const uint4 *vs = reinterpret_cast<const uint4 *>(a.v_cb + (size_t)h * (cb_bytes / 2));
    uint4 kst = make_uint4(0, 0, 0, 0), vst = kst;
    if (!REP && tid < n16) {
        kst = ks[tid];
        vst = vs[tid];
    }
    // 2. codes of the first two tiles, and q as the A operands of the four MFMAs: channels
    //    32 g + 8 i .. + 7 (the same for every row of the operand)
    uint32_t kA[NS][CW] = {}, vA[NS][CW] = {}, kB[NS][CW] = {}, vB[NS][CW] = {};
    half8_t qop[4] = {};
    if (active) {
        load_codes(k_base, 0, kA);
        load_codes(v_base, 0, vA);
        load_codes(k_base, 1, kB);
        load_codes(v_base, 1, vB);
#pragma unroll
        for (int i = 0; i < 4; ++i) qop[i] = ld16(a.q + (size_t)bh * D + 32 * g + 8 * i).h8;
    }
    constexpr int kNormWaves = 4;   // REP: wavefronts that look for the largest |entry|^2 of K, an entry per lane
    if constexpr (REP) {
        // 32 copies of every entry: consecutive lanes write consecutive 8-byte units (copy c = unit % 32 of entry
        // unit / 32); the 32 lanes of a copy set read one global address
        const uint2 *k8 = reinterpret_cast<const uint2 *>(ks), *v8 = reinterpret_cast<const uint2 *>(vs);
        // (all loads first: taken one unit at a time, each waits out a round trip to L2)
        constexpr int kPer = 256 * kAttnRepCopies / (kAttnWaves * 64 * SEQ), kStep = kAttnWaves * 64 * SEQ;
        uint2 ke[kPer], ve[kPer];
        const uint2 kn = k8[min(tid, a.E - 1)];
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int e = min((tid + i * kStep) / kAttnRepCopies, a.E - 1);
            ke[i] = k8[e];
            ve[i] = v8[e];
        }
#pragma unroll
        for (int i = 0; i < kPer; ++i) {   // (past the end of a smaller codebook: copies of its last entry, never read)
            reinterpret_cast<uint2 *>(smem)[tid + i * kStep] = ke[i];
            reinterpret_cast<uint2 *>(smem + kAttnRepSide)[tid + i * kStep] = ve[i];
        }
        if (wid < kNormWaves) {
            float n = 0.f;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const half2_t x = __builtin_bit_cast(half2_t, j ? kn.y : kn.x);
                n = __builtin_fmaf((float)x[0], (float)x[0], n);
                n = __builtin_fmaf((float)x[1], (float)x[1], n);
            }
            n = wave_max_uniform(n <= FLT_MAX ? n : INFINITY);   // (a NaN counts as infinity)
            if (lane == 0) norms[wid] = n;
        }
    } else {
        if (tid < n16) {
            reinterpret_cast<uint4 *>(smem)[tid] = kst;
            reinterpret_cast<uint4 *>(smem + v_off)[tid] = vst;
        }
        for (int i = tid + (int)blockDim.x; i < n16; i += (int)blockDim.x) {  // larger codebooks
            reinterpret_cast<uint4 *>(smem)[i] = ks[i];
            reinterpret_cast<uint4 *>(smem + v_off)[i] = vs[i];
        }
    }
    __syncthreads();
    // REP: no score is larger than |sm_scale log2 e| sum_p |q_p| max |entry|, and that not than |..| sqrt(P) |q| max |entry|.  Up to 60 (N(0, 1)
    // keys and queries of 128 channels: 32) the weights 2^score and their sums stay well inside fp32 without a running maximum
    // to subtract: the same relative precision, without the chain of maximum, comparison and branch between a tile's scores and
    // its weights.  B16 H32 T4096: 34.1 -> 33.2 us from HBM.  (Where the gathers of a shared copy set the pace it gives nothing, and a short
    // range pays for the bound: 300 tokens 8.1 -> 8.3.)
    bool fixed = false;
    if constexpr (REP) {
        float q2 = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) q2 = __builtin_fmaf((float)qop[i][j], (float)qop[i][j], q2);
        q2 += __shfl_xor(q2, 16, 64);
        q2 += __shfl_xor(q2, 32, 64);
        const float n2 = wave_max_uniform(norms[lane & (kNormWaves - 1)]);
        fixed = __builtin_amdgcn_readfirstlane(a.scale2 * a.scale2 * P * q2 * n2 <= 3600.f);
    }
    unsigned sh = SH;
    asm("" : "+v"(sh));
    // codebook of code position g CB + c (c < CB, all powers of two: (g CB + c) >> pg_shift is (g CB >> pg_shift) +
    // (c >> pg_shift)): a part of the lane's and one of the position's
    const unsigned lane_k = ((unsigned)((g * CB) >> a.pg_shift) * a.E) << SH, lane_v = (unsigned)v_off + lane_k;
    auto c_off = [&](int c) {   // a scalar, kept out of sight so that the sums are not all held in registers
        unsigned o = ((unsigned)(c >> a.pg_shift) * a.E) << SH;
        asm volatile("" : "+s"(o));
        return o;
    };
    // gathers of one group: the CB entries of step s, into a 64-byte register block in channel order
    // REP: lane constants of the two sides, byte 0 = 8 (lane % 32), byte 2 = the side's base / 65536
    const unsigned rep_k = (unsigned)(lane & 31) * 8u, rep_v = rep_k + (unsigned)kAttnRepSide;
    auto gather = [&](const uint32_t (&codes)[NS][CW], int s, int base, V16 (&blk)[4]) {
        if (!ONE) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            const unsigned w = codes[s][c / 4];
            if constexpr (REP) {
                // address bytes: [lane constant b0][code][lane constant b2][0]
                const unsigned sel = 0x0c020000u | ((4u + (unsigned)(c % 4)) << 8);
                lds_entry_into<V>(blk, c * V * 2, __builtin_amdgcn_perm(w, base ? rep_v : rep_k, sel));
                continue;
            }
            unsigned off = (c % 4) == 0 ? byte_shl<0>(w, sh)
                           : (c % 4) == 1 ? byte_shl<1>(w, sh)
                           : (c % 4) == 2 ? byte_shl<2>(w, sh) : byte_shl<3>(w, sh);
            if (!ONE) off += (base ? lane_v : lane_k) + c_off(c);
            lds_entry_into<V>(blk, c * V * 2, ONE ? (unsigned)base + off : off);
        }
    };

    float acc[32];  // channels 32 g .. 32 g + 31 of sum_t p_t V[t]
#pragma unroll
    for (int d = 0; d < 32; ++d) acc[d] = 0.f;
    float lsum = 0.f;          // per lane (every token is counted by its four lanes)
    // wave-uniform running maximum of the scores (log2 domain): finite, so that a masked token's weight is 2^-infinity = 0
    float m_run = REP && fixed && active ? 0.f : -FLT_MAX;

    V16 eb[2][4];  // entries of the group being used and of the one in flight
    gather(kA, 0, 0, eb[0]);  // (codes are zero when there is nothing to attend: entry 0, unused)

    // kn: K codes of the following tile (the other register buffer)
    auto tile_step = [&](int it, uint32_t (&kc)[NS][CW], uint32_t (&vc)[NS][CW], const uint32_t (&kn)[NS][CW]) {
        // scores.  Masked tokens get -inf through an additive bias (a select on the finished score
        // would make the compiler branch around the arithmetic and move the gathers).
        float sc[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (s + 1 < NS)
                gather(kc, s + 1, 0, eb[(s + 1) & 1]);
            else
                gather(vc, 0, v_off, eb[NS & 1]);
            if (NS == 1 || s + 2 == NS) load_codes(k_base, it + 2, kc);  // the K codes of this tile are used up
            float4_t c4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < 4; ++i) c4 = __builtin_amdgcn_mfma_f32_16x16x32_f16(qop[i], eb[s & 1][i].h8, c4, 0, 0, 0);
            const float bias = (t_lane + it * TILE + s * 16 < count) ? 0.f : -INFINITY;
            sc[s] = __builtin_fmaf(c4[0], a.scale2, bias);
        }
        // online softmax: raise the wave's running maximum if needed (uniform branches)
        if (!REP || !fixed) {
            float tmax = sc[0];
#pragma unroll
            for (int s = 1; s < NS; ++s) tmax = fmaxf(tmax, sc[s]);
            tmax = wave_max_uniform(tmax);
            if (tmax > m_run) {
                const float f = __builtin_amdgcn_exp2f(m_run - tmax);  // 0 while nothing was accumulated
#pragma unroll
                for (int d = 0; d < 32; ++d) acc[d] *= f;
                lsum *= f;
                m_run = tmax;
            }
        }

        // acc += p_t * V[t] on the lane's 32 channels
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (s + 1 < NS)
                gather(vc, s + 1, v_off, eb[(NS + s + 1) & 1]);
            else
                gather(kn, 0, 0, eb[0]);  // first K group of the next tile (2 NS is even)
            if (NS == 1 || s + 2 == NS) load_codes(v_base, it + 2, vc);
            const float p_t = __builtin_amdgcn_exp2f(sc[s] - m_run);
            lsum += p_t;
            const V16 (&ev)[4] = eb[(NS + s) & 1];
#pragma unroll
            for (int d = 0; d < 32; ++d) acc[d] += p_t * (float)ev[d / 8].h8[d % 8];
        }
    };
    for (int it = 0; it < ntiles; it += 2) {
        tile_step(it, kA, vA, kB);
        if (it + 1 < ntiles) tile_step(it + 1, kB, vB, kA);
    }

    // ---- reduce over the 16 token lanes, then over the wavefronts (fixed order) -------------
    row_reduce_scatter(acc, lane);
    lsum = wave_sum(lsum) * 0.25f;  // four lanes per token
    xw[wave * D + 32 * g + 2 * tok] = acc[0];
    xw[wave * D + 32 * g + 2 * tok + 1] = acc[1];
    if (lane == 0) {
        xw_m[wave] = m_run;
        xw_l[wave] = lsum;
    }
    __syncthreads();
    if (valid && tid - seq * (kAttnWaves * 64) < D) {
        const int d = tid - seq * (kAttnWaves * 64);
        float M = xw_m[0];
#pragma unroll
        for (int w = 1; w < kAttnWaves; ++w) M = fmaxf(M, xw_m[w]);
        float L = 0.f, o = 0.f;
#pragma unroll
        for (int w = 0; w < kAttnWaves; ++w) {
            float wgt = exp2f(xw_m[w] - M);   // (nothing attended: 2^(-FLT_MAX - M), or 1 where that goes for all; its sums are 0)
            L += xw_l[w] * wgt;
            o += xw[w * D + d] * wgt;
        }
        if (a.S == 1) {
            a.out[(size_t)bh * D + d] = (half_t)(L > 0.f ? o / L : 0.f);
        } else {
            float *wp = a.ws + ((size_t)bh * a.S + split) * (D + 2);
            wp[d] = o;
            if (d == 0) {
                wp[D] = M;
                wp[D + 1] = L;
            }
        }
    }
}

// Merge of the token-range partials by log-sum-exp (base 2), one workgroup per (b, h).  A launch of loads that take a trip to
// memory each: eight ranges are requested at once.  Attention of B3 H32 T3001, 32 codebooks (4 ranges)
// 16.7 -> 15.2 us with that, B1 H8 T30000 (59 ranges) 20.9 -> 17.7.
__global__ __launch_bounds__(128) void attn_merge_kernel(const float *__restrict__ ws, half_t *__restrict__ out,
                                                         int S) {
    constexpr int D = 128, N = 8;
    const int bh = blockIdx.x, d = threadIdx.x;
    const float *wp = ws + (size_t)bh * S * (D + 2);
    float m[N], l[N], x[N];
    auto request = [&](int s0) {   // (past the end: the last range once more)
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const float *p = wp + min(s0 + i, S - 1) * (D + 2);
            m[i] = p[D];
            l[i] = p[D + 1];
            x[i] = p[d];
        }
    };
    request(0);
    float M = m[0];
#pragma unroll
    for (int i = 1; i < N; ++i) M = fmaxf(M, m[i]);
    for (int s = N; s < S; s += N) {   // more than eight: the maximum of them all first
        float t[N];
#pragma unroll
        for (int i = 0; i < N; ++i) t[i] = wp[min(s + i, S - 1) * (D + 2) + D];
#pragma unroll
        for (int i = 0; i < N; ++i) M = fmaxf(M, t[i]);
    }
    float L = 0.f, o = 0.f;
    for (int s = 0; s < S; s += N) {
        if (s > 0) request(s);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if (s + i >= S) break;
            const float wgt = exp2f(m[i] - M);
            L += l[i] * wgt;
            o += x[i] * wgt;
        }
    }
    out[(size_t)bh * D + d] = (half_t)(L > 0.f ? o / L : 0.f);
}

// Token-range split: enough workgroups to fill the chip (two per compute unit) when batch x heads
// alone does not, ranges of at least kAttnMinTokens tokens, rounded to whole tiles.
//
// Codebooks so large that one workgroup fills a CU's LDS (G > 1): no more ranges than that, but the split and the items
// per workgroup (*seq) with the least estimated time.  Staging the codebooks costs a workgroup about two tiles' time, a
// tile 0.65 with one item on the CU, the merge launch 1.2; workgroups beyond 256 are another round.  (B = 3, H = 32,
// T = 3001, 32 codebooks per head and side: 6 ranges in 384 workgroups 22 us, 4 ranges in 192 17 us.)
static void attn_split(const vq_kv_t *kv, int *S, int *tc, int *seq) {
    const int tile = attn_tile(kv->v);
    const long long bh = (long long)kv->B * kv->H;
    long long want = bh > 0 ? (kAttnTargetWgs + bh - 1) / bh : 1;
    long long most = (kv->T + kAttnMinTokens - 1) / kAttnMinTokens;
    long long s = want < most ? want : most;
    if (s < 1) s = 1;
    auto range = [&](long long n) { return ((kv->T + n - 1) / n + tile - 1) / tile * tile; };   // tokens per range
    *seq = 1;
    const size_t side = (size_t)kv->cb_groups * kv->n_entries * kv->v * sizeof(half_t);
    if (kv->cb_groups > 1 && 2 * (2 * side + 4200) > 160 * 1024) {
        double best = 1e300;
        long long pick = s;
        for (long long n = s; n >= 1; --n)
            for (int q = 1; q <= 2; ++q) {
                if (q == 2 && kv->B * n < 2) continue;
                const long long wgs = (kv->B * n + q - 1) / q * kv->H, rounds = (wgs + 255) / 256;
                const double cost = rounds * (2.0 + (q == 2 ? 1.0 : 0.65) * (range(n) / tile)) + (n > 1 ? 1.2 : 0.0);
                if (cost < best) {
                    best = cost;
                    pick = n;
                    *seq = q;
                }
            }
        s = pick;
    }
    long long per = range(s);
    if (per < tile) per = tile;
    *tc = (int)per;
    *S = (int)((kv->T + per - 1) / per);
    if (*S < 1) *S = 1;
}

size_t attn_decode_workspace(const vq_kv_t *kv) {
    int S, tc, seq;
    attn_split(kv, &S, &tc, &seq);
    if (S == 1) return 0;
    return (size_t)kv->B * kv->H * S * (kv->D + 2) * sizeof(float);
}

template <int V, bool ONE, int SEQ, bool REP = false>
static int run_attn_seq(const AttnArgs &a, hipStream_t s) {
    const size_t side = REP ? (size_t)kAttnRepSide : ONE ? 4096 : (size_t)a.G * a.E * V * sizeof(half_t);  // matches the kernel's layout
    const size_t lds = 2 * side + (REP ? 16 * sizeof(float) : 0) + (size_t)SEQ * kAttnWaves * (128 + 2) * sizeof(float);
    // the kernel forms absolute LDS addresses: refused here, with an error, if it ever had static LDS
    static KernelSetup setup;
    if (int st = kernel_setup(reinterpret_cast<const void *>(&attn_decode_kernel<V, ONE, SEQ, REP>), lds, true, setup)) return st;
    const dim3 grid = SEQ == 1 ? dim3(a.B * a.H, a.S) : dim3((a.B * a.S + SEQ - 1) / SEQ * a.H);
    attn_decode_kernel<V, ONE, SEQ, REP><<<grid, kAttnWaves * 64 * SEQ, lds, s>>>(a);
    if (a.S > 1) attn_merge_kernel<<<a.B * a.H, 128, 0, s>>>(a.ws, a.out, a.S);
    return launch_status();
}

// Replicated codebooks: no bank conflicts, but 128 KiB to fill and only one workgroup (two items) per CU.  Worth it for long
// ranges in whole rounds of workgroups, and where a shared copy has conflicts (many entries).  H = 32 unless said, 256 entries,
// us, shared copy / copies: 16 x 4096 tokens 31.6 / 30.1, 16 x 8192 56.6 / 54.1, 8 x 16000 58.2 / 55.1; B32 H8 8192 34.6 / 33.4; but 16 x
// 3001 26.4 / 26.6, 16 x 300 8.3 / 10.2, 32 x 64 10.6 / 16.0, 5 x 16000 (320 workgroups) 46.2 / 58.7, 3 x 4096 17.6 / 24.0; 64 entries, 16 x
// 4096 29.5 / 29.8.  (S, tc: attn_split)
static bool attn_copies(const vq_kv_t *kv, int S, int tc) {
    const long long items = (long long)kv->B * S, wgs = (items + 1) / 2 * kv->H, rounds = (wgs + 255) / 256;
    return kv->cb_groups == 1 && kv->v == 4 && kv->n_entries > 128 && tc >= 4096 && items >= 2 && 20 * wgs >= 19 * 256 * rounds;
}

bool attn_replicated(const vq_kv_t *kv) {
    int S, tc, seq;
    attn_split(kv, &S, &tc, &seq);
    return attn_copies(kv, S, tc);
}

template <int V, bool ONE>
static int run_attn(const AttnArgs &a, int seq, bool copies, hipStream_t s) {
    if constexpr (!ONE)
        if (seq == 2) return run_attn_seq<V, false, 2>(a, s);
    if constexpr (ONE && V == 4)
        if (copies) return run_attn_seq<4, true, 2, true>(a, s);
    return run_attn_seq<V, ONE, 1>(a, s);
}

int launch_attn_decode(const vq_kv_t *kv, const void *q, float sm_scale, void *out, void *ws, hipStream_t s) {
    if (kv->D != 128) return VQ_ERR_UNSUPPORTED;
    if ((kv->cb_groups * kv->n_entries * kv->v) % 8 != 0) return VQ_ERR_UNSUPPORTED;  // 128-bit codebook staging
    AttnArgs a;
    a.k_codes = (const uint8_t *)kv->k_codes;
    a.v_codes = (const uint8_t *)kv->v_codes;
    a.k_cb = (const half_t *)kv->k_codebooks;
    a.v_cb = (const half_t *)kv->v_codebooks;
    a.seq_lens = kv->seq_lens;
    a.q = (const half_t *)q;
    a.out = (half_t *)out;
    a.ws = (float *)ws;
    a.B = kv->B;
    a.H = kv->H;
    a.T = kv->T;
    a.E = kv->n_entries;
    a.G = kv->cb_groups;
    int seq;
    attn_split(kv, &a.S, &a.tc, &seq);
    a.scale2 = sm_scale * kLog2e;
    {
        int pg = (kv->D / kv->v) / kv->cb_groups, sh = 0;
        while ((1 << sh) < pg) ++sh;
        if ((1 << sh) != pg) return VQ_ERR_UNSUPPORTED;
        a.pg_shift = sh;
    }
    const bool one = kv->cb_groups == 1, copies = attn_copies(kv, a.S, a.tc);
    if (kv->v == 8) return one ? run_attn<8, true>(a, seq, copies, s) : run_attn<8, false>(a, seq, copies, s);
    if (kv->v == 4) return one ? run_attn<4, true>(a, seq, copies, s) : run_attn<4, false>(a, seq, copies, s);
    return one ? run_attn<2, true>(a, seq, copies, s) : run_attn<2, false>(a, seq, copies, s);
}

}  // namespace vq
