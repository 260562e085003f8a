// VQ-gemv at batch size 1 for LONG lists of weights with small codebooks (uint8 codes, v = 8, one or two additive
// codebooks of <= 256 entries), one launch: products of x with every codebook entry are formed once and looked up.
// Operation: VQ-LLM (arXiv 2503.02236) Sec. III-C "VQ-gemv" at bs = 1, residual codebooks as in Sec. II-A.  (That the
// inner product of x with an entry is the same for every row that holds its code is the paper's Sec. II-A property of
// vector quantization turned around.)
//
// What it does.  y[n] = scale[n] sum_j sum_r C_r[code] . x_j.  For a slice of 64 sub-vector positions j the 2 x 256 x 64
// products C_r[e] . x_j are a table of 128 KiB fp32, which fits the LDS of a compute unit; a code then costs one 4-byte
// read and one addition, where gathering the entry costs a 16-byte read and four v_dot2 (gemv_replica.hip: 130 issue
// slots per 1024 codes and wavefront, 8 per 64 codes; here 3.4).
//   The table is a matrix product, [512 entries x 8] x [8 x 64 positions]: one v_mfma_f32_32x32x16_f16 (half of its k
//   range idle) gives 32 entries x 32 positions, two per wavefront and slice.
//   Table layout: entry e of codebook r at r * 64 KiB + e * 256, position 8 q + j of the slice in column 32 (j / 4) + 4 q +
//   j % 4 of the 64 four-byte columns.  LDS serves 32 lanes at a time and has 32 banks for 4-byte reads: lanes whose
//   columns differ modulo 32 never collide, whatever the codes are (0.97 ns per wavefront and read; 1.75 when two
//   lanes share a bank, 2.8 at random).
//
// Mapping.  One persistent workgroup of 16 wavefronts per compute unit.  A segment is a run of rows of one problem with
// all its slices; the host deals segments so that every workgroup gets the same share of the list.  Step i of a slice
// reads 128 rows, eight per wavefront: lane (row = lane / 8, q = lane % 8) loads the 16 code bytes of positions
// [8 q, 8 q + 8) of its row, so 128 bytes of every row and whole lines.  Lookup t of a step must find the lanes of four rows (32
// lanes) at different positions: row takes its positions in the order t ^ (row % 4) -- the low bit by the byte that the
// address permute picks (a per-lane selector), the next by swapping neighbouring dwords.  The lanes of a row are added by
// three DPP steps and one lane adds the sum to the row's accumulator in LDS (one wavefront and lane per row, in slice
// order: every order is fixed, and a row's bits do not depend on how the list was dealt over the workgroups).
// A ring of eight steps' codes is in flight per wavefront (128 KiB per compute unit), across slices, segments and problems;
// the barriers around a table wait for LDS traffic only.  R = 1: a slice has 128 positions, even ones in the first half of
// the table and odd ones in the second, and everything else is the same.
//
// Bound: memory.  32 decoder blocks of Llama-7B shape, two codebooks (224 problems, 1.63 GB): 282 us, 5.8 TB/s, where
// gathering entries takes 463 - 481; with the lookups switched off 270 us, with all codes from cache 195 us.  Counters: vector
// issue 55 % of the launch, LDS 50 % (0.5 % of that conflicts), 1.68 GB read.
#include <algorithm>
#include <new>
#include <vector>

#include "vq_common.h"

namespace vq {

constexpr int kLutThreads = 1024;
constexpr int kLutWaves = kLutThreads / kWave;
constexpr int kLutTable = 2 * 65536;                  // LDS bytes of the table
constexpr int kLutLds = 160 * 1024;
constexpr int kLutRing = 8;                           // steps in flight per wavefront
constexpr int kLutStepRows = kLutWaves * 8;           // rows of a step

// A run of rows of one problem: every every-th row, so that all of them lie alike in their 128-byte lines (see lut_subs).
struct LutSegment {
    const uint8_t *codes;   // the line in which its first row starts, `lead` bytes into it
    const half_t *cb;       // [R][E][8]
    const half_t *scale;    // of its first row, or null
    const half_t *x;        // [K]
    half_t *y;              // of its first row
    int rows, K, E;
    int steps;              // steps per slice: ceil(rows / kLutStepRows)
    int slices;
    int stride;             // bytes from row to row of the segment
    int lead;
    int every;
};
static_assert(sizeof(LutSegment) == 72, "table layout");

__device__ __forceinline__ void lut_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

typedef __attribute__((address_space(3))) float lds_f32_t;
typedef uint32_t lut_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t lut_u32x2 __attribute__((ext_vector_type(2)));
// global memory by address space, so that the accesses are no generic ones (which would count as LDS accesses too)
#define VQ_GLOBAL(T, p) ((__attribute__((address_space(1))) T *)(p))

template <int CTRL>
__device__ __forceinline__ float lut_dpp_add(float x) {
    const int y = __builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true);
    return x + __int_as_float(y);
}

// The segment table lies in device memory and is read with scalar loads.
__device__ __forceinline__ LutSegment lut_segment(const LutSegment *table, int k) {
    const __attribute__((address_space(4))) uint64_t *q =
        (const __attribute__((address_space(4))) uint64_t *)(uintptr_t)(table + k);
    LutSegment s;
    s.codes = (const uint8_t *)q[0];
    s.cb = (const half_t *)q[1];
    s.scale = (const half_t *)q[2];
    s.x = (const half_t *)q[3];
    s.y = (half_t *)q[4];
    const uint64_t a = q[5], b = q[6], c = q[7], d = q[8];
    s.rows = (int)(uint32_t)a; s.K = (int)(a >> 32);
    s.E = (int)(uint32_t)b; s.steps = (int)(b >> 32);
    s.slices = (int)(uint32_t)c; s.stride = (int)(c >> 32);
    s.lead = (int)(uint32_t)d; s.every = (int)(d >> 32);
    return s;
}

template <int R>
__global__ __launch_bounds__(kLutThreads) void gemv_lut_kernel(const LutSegment *table, const int *first) {
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int seg0 = first[blockIdx.x], seg1 = first[blockIdx.x + 1];
    if (seg0 >= seg1) return;
    constexpr int kSliceBytes = 128;                  // of a row's codes
    const int row = lane >> 3, q = lane & 7;
    const bool odd = row & 1, swap = row & 2;
    // address bytes of lookup t = 2 d + i of a step: [4 * column][code][table half][0]; the columns of dword d and the
    // constants 1 and 0 in kc[d], the lane's choice of code byte in sel[i][r]
    uint32_t kc[4], sel[2][2];
    const uint32_t pick = swap ? 0x07060504u : 0x03020100u;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const uint32_t od = (uint32_t)(swap ? d ^ 1 : d);   // dword of the lane's 16 bytes that comes d-th
        const uint32_t c0 = 32u * (od >> 1) + 4u * q + 2u * (od & 1u);   // column of its first position
        const uint32_t p0 = 4u * (c0 + (odd ? 1u : 0u)), p1 = 4u * (c0 + (odd ? 0u : 1u));
        kc[d] = p0 | (p1 << 8) | 0x00010000u;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const uint32_t byte = 2u * (odd ? 1u - i : (uint32_t)i) + r;
            sel[i][r] = (4u + i) | (byte << 8) | ((r ? 6u : 7u) << 16) | 0x0C000000u;
        }

    // ---- requests: the codes of step i of slice s of a segment, kLutRing steps in front of the work
    // (Ordinary loads: the compiler keeps their registers and counts them, vmcnt(7) in front of every step, also around the loop
    // and past a new table.  With the same loads and waits as asm 280.4 us for the 32-block stack, here 281.4.)
    struct Codes {
        lut_u32x4 v;        // R = 2
        lut_u32x2 lo, hi;   // R = 1
    };
    Codes ring[kLutRing];
    // A slice is a whole number of turns of the ring (past its last step the slots hold the last row once more), so the
    // requests of a turn all belong to one slice: `rq` is the turn after the one that is worked on.
    int rq_seg = seg0, rq_slice = 0, rq_turn = 0;   // rq_turn: its first step
    uint32_t rq_col, rq_off;            // lane: its chunk of a row, and with its row of a step
    uint32_t rq_second;                 // R = 1: from its first 8 bytes to the other 8
    const uint8_t *rq_base;             // codes of the turn's first row
    LutSegment rq = lut_segment(table, rq_seg);
    // Whether byte `at` of the segment's lines belongs to its row.
    auto inside = [](const LutSegment &g, int at) { return at >= g.lead && at < g.lead + (g.K >> 3) * R; };
    auto rq_slice_start = [&]() {
        rq_turn = 0;
        rq_base = rq.codes;
        const int at = rq_slice * kSliceBytes + q * 16;
        // (a lane before the row or past it, or one half of it where R = 1, reads the row's first codes; what it looks up
        // is dropped)
        rq_col = inside(rq, at) ? at : rq.lead;
        rq_second = (inside(rq, at + 8) ? at + 8 : rq.lead) - rq_col;
        rq_off = rq_col + (uint32_t)((8 * wave + row) * rq.stride);
    };
    rq_slice_start();
    auto load = [&](Codes &c, const uint8_t *base, uint32_t off) {
        if constexpr (R == 2) {
            c.v = __builtin_nontemporal_load((const __attribute__((address_space(1))) lut_u32x4 *)(base + off));
        } else {
            c.lo = __builtin_nontemporal_load((const __attribute__((address_space(1))) lut_u32x2 *)(base + off));
            c.hi = __builtin_nontemporal_load((const __attribute__((address_space(1))) lut_u32x2 *)(base + (off + rq_second)));
        }
    };
    // Request of slot t of the turn `rq`: rows past the segment's last are that row.
    auto request = [&](Codes &c, int t) {
        const int last = rq.rows - 1 - rq_turn * kLutStepRows;      // of the turn's rows (>= 0: a turn starts with a row)
        const int r0 = t * kLutStepRows + 8 * wave;
        const uint8_t *base = rq_base + (size_t)(uint32_t)(t * kLutStepRows) * (uint32_t)rq.stride;
        uint32_t off = rq_off;
        if (r0 + 7 > last) {                                        // (uniform)
            asm volatile("");                                       // (a branch: not worth five instructions every time)
            base = rq_base;
            off = rq_col + (uint32_t)min(r0 + row, last) * (uint32_t)rq.stride;
        }
        load(c, base, off);
    };
    auto rq_next = [&]() {
        rq_turn += kLutRing;
        rq_base += (size_t)(uint32_t)(kLutRing * kLutStepRows) * (uint32_t)rq.stride;
        if (rq_turn < rq.steps) return;
        if (++rq_slice == rq.slices) {
            if (rq_seg + 1 == seg1) {    // nothing left: the same turn again, in cache
                --rq_slice;
            } else {
                rq = lut_segment(table, ++rq_seg);
                rq_slice = 0;
            }
        }
        rq_slice_start();
    };
#pragma unroll
    for (int t = 0; t < kLutRing; ++t) request(ring[t], t);
    rq_next();

    // ---- work
    const int ln = lane & 31, lh = lane >> 5;
    LutSegment sg;
    half8_t ent;                        // A operand: 32 entries of the wavefront (codebook wave / 8, entries 32 (wave % 8) ..)
    int seg = seg0, slice = 0;
    bool whole = true;                  // the slice lies in the row
    bool in_row[2] = {true, true};      // the halves of the lane's chunk do (R = 2: both or none)
    lds_f32_t *acc = nullptr;           // row sums of the segment, behind x
    lds_f32_t *acc_lane = nullptr;      // where the lane's current row lies

    // Entries and x of the next segment.  (Requested here and waited for: two or three times per workgroup.)
    auto segment_start = [&]() {
        sg = lut_segment(table, seg);
        const int e = min(32 * (wave & 7) + ln, sg.E - 1) + (R == 2 && wave >= 8 ? sg.E : 0);
        const lut_u32x4 ev = VQ_GLOBAL(const lut_u32x4, sg.cb)[e];
        // sub-vectors of x, zeros before them and up to the last slice's end
        const int xunits = sg.K >> 3, before = sg.lead / R, xend = sg.slices * (R == 2 ? 64 : 128);
        for (int u = tid; u < xend; u += kLutThreads) {
            lut_u32x4 v = {0, 0, 0, 0};
            if (u >= before && u < before + xunits) v = VQ_GLOBAL(const lut_u32x4, sg.x)[u - before];
            *(__attribute__((address_space(3))) lut_u32x4 *)(uintptr_t)(kLutTable + u * 16) = v;
        }
        acc = (lds_f32_t *)(uintptr_t)(kLutTable + xend * 16);
        for (int r = tid; r < sg.rows; r += kLutThreads) acc[r] = 0.f;
        V16 a;
        a.u = lh ? make_uint4(0, 0, 0, 0) : make_uint4(ev.x, ev.y, ev.z, ev.w);
        ent = a.h8;
        lut_barrier();
    };
    // The table of the current slice; every wavefront is done with the one before it.
    auto build = [&]() {
        const int s = slice;
        lds_f32_t *dst = (lds_f32_t *)(uintptr_t)((wave >> 3) * 65536 + (32 * (wave & 7) + 4 * lh) * 256 + ln * 4);
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) {
            const int p = 8 * (ln >> 2) + 4 * ct + (ln & 3);   // position in column 32 ct + ln
            const int u = R == 2 ? s * 64 + p : s * 128 + 2 * p + (wave >> 3);
            const lut_u32x4 t = *(__attribute__((address_space(3))) lut_u32x4 *)(uintptr_t)(kLutTable + u * 16);
            V16 v;
            v.u = lh ? make_uint4(0, 0, 0, 0) : make_uint4(t.x, t.y, t.z, t.w);
            const float16_t zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            const float16_t d = __builtin_amdgcn_mfma_f32_32x32x16_f16(ent, v.h8, zero, 0, 0, 0);
#pragma unroll
            for (int j = 0; j < 16; ++j) dst[(8 * (j >> 2) + (j & 3)) * 64 + ct * 32] = d[j];
        }
        lut_barrier();
        const int at = s * kSliceBytes;
        whole = inside(sg, at) && inside(sg, at + kSliceBytes - 1);
        in_row[0] = inside(sg, at + q * 16);
        in_row[1] = R == 1 ? inside(sg, at + q * 16 + 8) : in_row[0];
        acc_lane = acc + 8 * wave + row;
    };
    auto step = [&](const Codes &c, lds_f32_t *sum) {
        uint32_t in[4], w[4];
        if constexpr (R == 2) {
            in[0] = c.v.x; in[1] = c.v.y; in[2] = c.v.z; in[3] = c.v.w;
        } else {
            in[0] = c.lo.x; in[1] = c.lo.y; in[2] = c.hi.x; in[3] = c.hi.y;
        }
#pragma unroll
        for (int d = 0; d < 4; ++d) w[d] = __builtin_amdgcn_perm(in[d ^ 1], in[d], pick);   // (a byte permute as a select)
        float v[16];
        const float so_far = *sum;   // (an LDS float atomic instead of this read and the write below: 24 clocks, not 4)
#pragma unroll
        for (int t = 0; t < 8; ++t)
#pragma unroll
            for (int r = 0; r < 2; ++r)
                v[2 * t + r] = *(lds_f32_t *)(uintptr_t)__builtin_amdgcn_perm(kc[t >> 1], w[t >> 1], sel[t & 1][r]);
        if (R == 1 && !whole) {      // (uniform; not by a zero of x: the row's first code may name an infinity)
#pragma unroll
            for (int t = 0; t < 16; ++t) v[t] = in_row[t >> 3] ? v[t] : 0.f;
        }
        float s0 = v[0], s1 = v[1];
#pragma unroll
        for (int t = 1; t < 8; ++t) {
            s0 += v[2 * t];
            s1 += v[2 * t + 1];
        }
        float s = s0 + s1;
        if (R == 2 && !whole) s = in_row[0] ? s : 0.f;
        s = lut_dpp_add<0xB1>(s);    // quad_perm [1,0,3,2]
        s = lut_dpp_add<0x4E>(s);    // quad_perm [2,3,0,1]
        s = lut_dpp_add<0x141>(s);   // row_half_mirror: all eight lanes of the row
        if (q == 0) *sum = so_far + s;
    };

    segment_start();
    build();
    while (true) {
        for (int i = 0; i < sg.steps; i += kLutRing) {
#pragma unroll
            for (int t = 0; t < kLutRing; ++t) {
                if (i + t < sg.steps) step(ring[t], acc_lane + t * kLutStepRows);
                request(ring[t], t);
            }
            acc_lane += kLutRing * kLutStepRows;
            rq_next();
        }
        lut_barrier();   // every wavefront is done with the table
        if (++slice == sg.slices) {
            for (int r = tid; r < sg.rows; r += kLutThreads) {
                const float sc = sg.scale ? (float)VQ_GLOBAL(const half_t, sg.scale)[r * sg.every] : 1.f;
                VQ_GLOBAL(half_t, sg.y)[r * sg.every] = (half_t)(acc[r] * sc);
            }
            if (++seg == seg1) return;
            lut_barrier();   // (the sums are read before they are cleared)
            slice = 0;
            segment_start();
        }
        build();
    }
}

namespace {

KernelSetup g_lut_setup[2];

constexpr int kLutMaxGrid = 256;

// The rows of a problem that lie alike in their 128-byte lines of codes, or all of them.  A slice must be whole lines: when
// rows are not a multiple of a line long, a slice of a row that starts inside a line would take two, and the neighbouring
// slice, minutes of traffic later, one of them again (K = 11008, two codebooks: 2752 bytes, 3.9 TB/s against 5.3 for
// K = 11264).  Every 128 / gcd(row, 128)-th row starts alike; they make a problem of their own with x shifted by the lead.
// Not for problems with few rows, where the extra tables cost more than the lines.
constexpr int kLutClassRows = 1024;
struct LutSub {
    int problem, cls, every;   // rows cls, cls + every, ...
    int rows, slices, lead;
    int cap;                   // rows per segment: their sums lie behind x in LDS
};
std::vector<LutSub> lut_subs(const std::vector<const vq_weight_t *> &w) {
    std::vector<LutSub> subs;
    for (int k = 0; k < (int)w.size(); ++k) {
        const int R = w[k]->n_codebooks, row_bytes = w[k]->K / 8 * R;
        int every = 1;
        while (every * row_bytes % 128) every *= 2;
        const bool split = w[k]->N / every >= kLutClassRows;
        if (!split) every = 1;
        for (int c = 0; c < every; ++c) {
            LutSub s;
            s.problem = k;
            s.cls = c;
            s.every = every;
            s.rows = (w[k]->N - c + every - 1) / every;
            s.lead = every * row_bytes % 128 ? 0 : (int)(((uintptr_t)w[k]->codes + (size_t)c * row_bytes) % 128);
            s.slices = (row_bytes + s.lead + 127) / 128;
            s.cap = (kLutLds - kLutTable - s.slices * (R == 2 ? 64 : 128) * 16) / 4 / kLutStepRows * kLutStepRows;
            subs.push_back(s);
        }
    }
    return subs;
}

// Deals the rows of all problems to at most `grid` workgroups, each up to `share` (in steps; building a slice's table
// counts like kLutBuild of a step).  pieces: in order; first[b]: first piece of workgroup b.
// Returns false if `share` is too small.
constexpr double kLutBuild = 0.75;
struct LutPiece {
    int sub, row0, rows;
};
bool lut_deal(const std::vector<LutSub> &subs, int grid, double share, std::vector<LutPiece> *pieces, std::vector<int> *first) {
    int b = 0, count = 0;
    double room = share;
    if (pieces) {
        pieces->clear();
        first->assign(1, 0);
    }
    for (int k = 0; k < (int)subs.size(); ++k) {
        const LutSub &u = subs[k];
        const int cap = u.cap / kLutStepRows;
        int row = 0;
        while (row < u.rows) {
            const int want = (u.rows - row + kLutStepRows - 1) / kLutStepRows;
            int n = (int)(room / u.slices - kLutBuild);
            n = std::min(std::min(n, cap), want);
            // (a stub of a segment at the end of a share is not worth its tables)
            if (n < 1 || (n < want && n < cap && n < 3 && room < share)) {
                if (room == share) return false;
                if (++b == grid) return false;
                if (pieces) first->push_back(count);
                room = share;
                continue;
            }
            const int rows = std::min(n * kLutStepRows, u.rows - row);
            if (pieces) pieces->push_back({k, row, rows});
            ++count;
            row += rows;
            room -= u.slices * (n + kLutBuild);
        }
    }
    if (pieces)
        while ((int)first->size() <= grid) first->push_back(count);
    return true;
}

double lut_share(const std::vector<LutSub> &subs, int grid) {
    double lo = 0, hi = 64;
    while (!lut_deal(subs, grid, hi, nullptr, nullptr)) hi *= 2;
    for (int i = 0; i < 30; ++i) {
        const double mid = 0.5 * (lo + hi);
        (lut_deal(subs, grid, mid, nullptr, nullptr) ? hi : lo) = mid;
    }
    return hi;
}

std::vector<const vq_weight_t *> lut_weights(const vq_gemv_call_t *calls, int n_calls) {
    std::vector<const vq_weight_t *> w;
    for (int c = 0; c < n_calls; ++c)
        for (int i = 0; i < calls[c].count; ++i) w.push_back(calls[c].w[i]);
    return w;
}

constexpr size_t kLutFirstBytes = ((kLutMaxGrid + 1) * sizeof(int) + 255) & ~(size_t)255;

}  // namespace

struct GemvLutList {
    int device, R, grid;
    const LutSegment *table;   // device
    const int *first;          // device
};

// Whether this kernel is the better one for a list (of weights of the kind gemv_replica_supported accepts): both times are
// estimated from the launch shapes.
//   Here a workgroup takes its segments one after the other; a slice costs kLutSliceUs (table, and codes that come a
//   memory latency after the previous slice's) or kLutStepUs per step, whichever is more.
//   gemv_replica.hip: a group of workgroups takes its problems one after the other, kRepProblemUs for each and kRepItemUs
//   per item (512 positions of a row) of a wavefront.
// Decoder blocks of Llama-7B shape, this kernel against that one, us: two codebooks, 1 block 55 / 26, 2 57 / 50, 4 66 / 84, 8 86 / 136,
// 32 278 / 475; half the width 1 block 31 / 16, 4 33 / 41, 32 89 / 205; an eighth 16 blocks 11 / 42.  One codebook, 3 blocks 48 / 58, 4
// 55 / 57, 8 70 / 81, 12 109 / 134, 32 186 / 291; half the width 3 blocks 26 / 30, 8 34 / 41, 32 69 / 136; a quarter 8 blocks 16 / 26; an
// eighth 11 / 18.  The estimates are good to a few per cent, and this kernel must be ahead by more (few rows and a long K: 100 x
// 512 x 12288, two codebooks, 68 / 64, 48 x 1024 x 11008 68 / 54): over 184 lists none that takes it is slower for it.  A list that is
// short both ways (kLutMinBytes of codes, kLutMinProblems) stays with that kernel, whose bits do not depend on the list.
constexpr double kLutMinBytes = 16 << 20, kLutStartUs = 6, kLutSegmentUs = 2, kLutSliceUs[2] = {3.9, 2.3}, kLutStepUs = 0.6;
constexpr int kLutMinProblems = 48;
constexpr double kRepStartUs = 4, kRepProblemUs = 3.5, kRepItemUs[2] = {0.6, 1.0};
bool gemv_lut_worth(const vq_gemv_call_t *calls, int n_calls) {
    const std::vector<const vq_weight_t *> w = lut_weights(calls, n_calls);
    const int n = (int)w.size(), R = w[0]->n_codebooks;
    double bytes = 0;
    for (const vq_weight_t *p : w) bytes += (double)p->N * (p->K / 8) * R;
    if (bytes < kLutMinBytes && n < kLutMinProblems) return false;
    const std::vector<LutSub> subs = lut_subs(w);
    std::vector<LutPiece> pieces;
    std::vector<int> first;
    if (!lut_deal(subs, kLutMaxGrid, lut_share(subs, kLutMaxGrid), &pieces, &first)) return false;
    double here = 0, there = 0;
    for (int b = 0; b < kLutMaxGrid; ++b) {
        double t = kLutStartUs;
        for (int i = first[b]; i < first[b + 1]; ++i)
            t += kLutSegmentUs + subs[pieces[i].sub].slices * std::max(kLutSliceUs[R - 1], kLutStepUs * ((pieces[i].rows + kLutStepRows - 1) / kLutStepRows));
        here = std::max(here, t);
    }
    int groups = 1;
    while (groups < 32 && groups * 2 <= n) groups *= 2;
    for (int g = 0; g < groups; ++g) {
        double t = kRepStartUs;
        for (int k = g; k < n; k += groups)
            t += kRepProblemUs + kRepItemUs[R - 1] * ((w[k]->N * groups + 255) / 256) * ((w[k]->K + 4095) / 4096) / 16;
        there = std::max(there, t);
    }
    return here < 0.95 * there;
}

// Segments: at most one more per workgroup than the problems need by themselves.
size_t gemv_lut_list_workspace(const vq_gemv_call_t *calls, int n_calls) {
    size_t segs = kLutMaxGrid;
    for (const LutSub &u : lut_subs(lut_weights(calls, n_calls))) segs += (u.rows + u.cap - 1) / u.cap;
    return kLutFirstBytes + ((segs * sizeof(LutSegment) + 255) & ~(size_t)255);
}

int gemv_lut_list_create(const vq_gemv_call_t *calls, int n_calls, void *ws, hipStream_t s, GemvLutList **out) {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        return VQ_ERR_LAUNCH;
    const int grid = std::min(cus, kLutMaxGrid);
    const std::vector<const vq_weight_t *> w = lut_weights(calls, n_calls);
    std::vector<const void *> x;
    std::vector<void *> y;
    for (int c = 0; c < n_calls; ++c)
        for (int i = 0; i < calls[c].count; ++i) {
            x.push_back(calls[c].x[i]);
            y.push_back(calls[c].y[i]);
        }
    const std::vector<LutSub> subs = lut_subs(w);
    std::vector<LutPiece> pieces;
    std::vector<int> first;
    if (!lut_deal(subs, grid, lut_share(subs, grid), &pieces, &first)) return VQ_ERR_LAUNCH;
    std::vector<LutSegment> table(pieces.size());
    for (size_t i = 0; i < pieces.size(); ++i) {
        const LutPiece &p = pieces[i];
        const LutSub &u = subs[p.sub];
        const vq_weight_t *pw = w[u.problem];
        const int row_bytes = pw->K / 8 * pw->n_codebooks;
        const size_t row = u.cls + (size_t)p.row0 * u.every;
        LutSegment &g = table[i];
        g.codes = (const uint8_t *)pw->codes + row * row_bytes - u.lead;
        g.cb = (const half_t *)pw->codebooks;
        g.scale = pw->scale ? (const half_t *)pw->scale + row : nullptr;
        g.x = (const half_t *)x[u.problem];
        g.y = (half_t *)y[u.problem] + row;
        g.rows = p.rows;
        g.K = pw->K;
        g.E = pw->n_entries;
        g.steps = (p.rows + kLutStepRows - 1) / kLutStepRows;
        g.slices = u.slices;
        g.stride = row_bytes * u.every;
        g.lead = u.lead;
        g.every = u.every;
    }
    if (kLutFirstBytes + table.size() * sizeof(LutSegment) > gemv_lut_list_workspace(calls, n_calls)) return VQ_ERR_LAUNCH;
    GemvLutList *h = new (std::nothrow) GemvLutList;
    if (!h) return VQ_ERR_LAUNCH;
    if (hipMemcpyAsync(ws, first.data(), (size_t)(grid + 1) * sizeof(int), hipMemcpyHostToDevice, s) != hipSuccess ||
        hipMemcpyAsync((unsigned char *)ws + kLutFirstBytes, table.data(), table.size() * sizeof(LutSegment), hipMemcpyHostToDevice, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess) {
        (void)hipGetLastError();
        delete h;
        return VQ_ERR_LAUNCH;
    }
    h->device = dev;
    h->R = w[0]->n_codebooks;
    h->grid = grid;
    h->first = (const int *)ws;
    h->table = (const LutSegment *)((unsigned char *)ws + kLutFirstBytes);
    *out = h;
    return VQ_OK;
}

void gemv_lut_list_destroy(GemvLutList *h) { delete h; }

int launch_gemv_lut_list(const GemvLutList *h, hipStream_t s) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != h->device) return VQ_ERR_LAUNCH;
    const void *fn = h->R == 2 ? (const void *)gemv_lut_kernel<2> : (const void *)gemv_lut_kernel<1>;
    if (int st = kernel_setup(fn, kLutLds, true, g_lut_setup[h->R - 1])) return st;
    if (h->R == 2) gemv_lut_kernel<2><<<h->grid, kLutThreads, kLutLds, s>>>(h->table, h->first);
    else gemv_lut_kernel<1><<<h->grid, kLutThreads, kLutLds, s>>>(h->table, h->first);
    return launch_status();
}

}  // namespace vq
