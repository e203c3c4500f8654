// All layers of a decode step of few requests in one launch (Eq. 3 and 4 over the whole stack; bf16 or 4-bit weights).
//
// With a few requests a layer is nine or ten launches of 5 to 40 us, and what they lose is what surrounds their steady state: the
// boundary (a launch costs 4 to 5 us beside its work), the first requests' latency, the drain.  Here one workgroup per
// compute unit stays for the whole stack and the phases of a layer
//   q/k/v -> attention -> merge -> o -> gate/up -> down
// are separated by a barrier over the grid (2.6 us from the last arrival's stores to the next phase's loads on 16 counters, 0.5 less on 64), in front of which
// every wave but one requests its first weights.  Bound by the weight stream in the long phases (gate/up 6.6 to 7 TB/s) and by
// chains of small loads and stores around them.  Steps of 8 layers, launch per operation -> this (us), 1 / 8 / 16 requests of 200 to 1200
// cached tokens: 8B shape bf16 1154 -> 879 / 1185 -> 968 / 1217 -> 1077, 4-bit at 1 / 4 / 8 817 -> 607 / 835 -> 640 / 837 -> 675; hidden
// 2048, ffn 8192 bf16 644 -> 400 / 666 -> 457 / 697 -> 566, 4-bit at 1 / 8 510 -> 332 / 538 -> 384; hidden 1024 440 -> 283 / 476 -> 328 /
// 494 -> 403, 403 -> 282 / 430 -> 333.  Eight rows are what an operand of the 4-bit products holds beside their low planes; with
// two rows a wave and an operand of 16 for each plane (and the barrier on 16 counters) 4-bit steps at 12 / 16 requests (4 layers, 8B shape) took 549 -> 552 / 524 -> 553;
// two operands of eight rows were not built.  Hence kLayersRows and kLayersRowsW4.
//
// Hand-over between workgroups.  Data that another workgroup reads in the same launch is stored through to memory (st_agent),
// and its storer waits for vmcnt before it counts itself as arrived.  Readers either pass their caches by (ld_agent: the residual
// stream, partial sums, attention's partials), or, where many read the same bytes (activation tiles, q, the new cache
// entries), load plainly from places that no cache holds: 128-byte lines are written by one workgroup only and not read before
// the barrier behind their writing, and the tiles of as many layers as there is room for lie beside one another (8B shape: 25
// layers at one row, four at 16); before they are written again the readers' caches are invalidated (an acquire fence at
// agent scope by one wave of each compute unit).  Fences on both sides of every barrier instead: 61 us a barrier of 256
// workgroups instead of 3.9 (one counter).
//
// All workgroups have to be resident at once: the launch is a cooperative one (19 us more than a plain launch).
#include <hip/hip_fp16.h>

#include <atomic>
#include <type_traits>

#include "attn_items.hpp"
#include "grid.hpp"
#include "kernels.hpp"

namespace sun {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8;
static_assert(kLayersRowsW4 <= kWaves && kLayersRows <= 2 * kWaves, "one row a wave with 4-bit weights, two otherwise");
constexpr int kBlock = 128;        // columns of a block
constexpr int kUnits = 256;         // work units a phase is cut into at most (one per compute unit)
constexpr int kLayersPerLaunch = 48;
// Words between the counters of two blocks' arrivals: side by side, 32 blocks' arrivals are on one line and are added one after the
// other.  8 layers of the 8B shape, 1 / 8 / 32 words apart: five 4-bit requests 663 / 655 / 656 us, one bf16 request 883 / 881 / 882, sixteen
// 1165 / 1165 / 1166; step_begin_kernel clears them all.
constexpr int kApart = 8;
constexpr int kBfRow = 512;         // bytes of 128 activations of one row: [32-wide step][plane][32] bf16
constexpr int kQRow = 384;          // the same as 16-bit fixed point: [step of 64][plane][octet of 16] int8, then (scale, sum)
constexpr int kQHalf = 256;         // each step of 64 with a scale of its own: [plane][octet of 16] int8, then (scale, sum)

struct LayerPtrs {
    const void *g1, *g2, *qn, *kn, *bq, *bk, *bv;
};

struct RopeAppend {
    const float* table;
    const int32_t *seq_lens, *page_tables;
    uint16_t* pool;
    int64_t k_base, k_layer, k_page, k_head, k_token, k_dim, v_base, v_layer, v_page, v_head, v_token, v_dim;
    int Hq, Hkv, max_pages, n_pages, has_norm, has_bias;
};

struct MatP {
    const char* w;
    const char* sz;
    size_t w_step, sz_step;         // from one layer to the next
    int K, S, nblk;                 // split along k, column blocks
    uint32_t* arrived;              // [nblk][kApart]
};

struct LayersArgs {
    LayerPtrs lp[kLayersPerLaunch];
    MatP qkv, o, gu, down;
    AttnArgs attn;                  // of layer 0
    RopeAppend rope;
    const void* g1_next;            // g1 of layer l1, if there is one
    float* x;
    float *ssq1, *ssq2;             // [hidden / 128][kLayersRows] sums of squares of the residual stream
    float* slab;
    alignas(32) uint32_t *counters, *lost;   // what a wait reads, side by side
    uint32_t polls;
    char *t1, *ta, *t2, *tu;        // activation tiles of layer 0 and their steps; `ring` layers have their own
    float* q;
    size_t h_step, a_step, u_step, q_step;
    int l0, l1, n_layers, ring, R, H, s_only;
    float eps;
};

// ---------------- activation tiles ----------------
__device__ __forceinline__ float gain_at(const void* g, int i) { return bf16_bits_to_f32(((const uint16_t*)g)[i]); }

// A wave stores 128 activations of one row, columns 2 lane and 2 lane + 1 of it from each lane.
template <bool W4>
__device__ __forceinline__ void store_tile128(char* tile, int R, int chunk, int row, float y0, float y1) {
    const int lane = lane_here();
    if constexpr (!W4) {
        char* p = tile + ((size_t)chunk * R + row) * kBfRow + (lane >> 4) * 128 + (lane & 15) * 4;
        uint16_t l0, l1;
        const uint32_t h0 = split_bf16(y0, l0), h1 = split_bf16(y1, l1);
        st_agent((uint32_t*)p, h0 | h1 << 16);
        st_agent((uint32_t*)(p + 64), (uint32_t)l0 | (uint32_t)l1 << 16);
    } else {
        char* p = tile + ((size_t)chunk * R + row) * kQRow;
        const float am = wave_max(fmaxf(fabsf(y0), fabsf(y1))), inv = qtile_inv(am);
        const int x0 = (int)rintf(y0 * inv), x1 = (int)rintf(y1 * inv);
        const int l0 = ((x0 + 128) & 255) - 128, l1 = ((x1 + 128) & 255) - 128;
        const uint32_t lo = (uint32_t)(l0 & 255) | (uint32_t)(l1 & 255) << 8;
        const uint32_t hi = (uint32_t)(((x0 - l0) >> 8) & 255) | (uint32_t)(((x1 - l1) >> 8) & 255) << 8;
        // four columns of a plane per lane: even lanes the high plane's, odd lanes the low plane's
        const uint32_t got = lane_xor<1>(lane & 1 ? hi : lo);
        const uint32_t v = lane & 1 ? (got | lo << 16) : (hi | got << 16);
        const int c = 4 * (lane >> 1), half = c >> 6, s = (c >> 4) & 3;
        st_agent((uint32_t*)(p + (((s & 1) * 2 + (lane & 1)) * 4 + half * 2 + (s >> 1)) * 16 + (c & 15)), v);
        const int sum = wave_sum(x0 + x1);
        if (lane == 0) st_agent2((float*)(p + 256), am / kQMax, __int_as_float(sum));
    }
}

// A wave stores 64 activations of one row, one from each lane: the lower or upper half of a 128-wide chunk.
__device__ __forceinline__ void store_tile64(char* tile, int R, int chunk, int upper, int row, float y) {
    const int lane = lane_here();
    uint16_t lo;
    const uint16_t hi = split_bf16(y, lo);
    const uint32_t got = lane_xor<1>((uint32_t)(lane & 1 ? hi : lo));
    const uint32_t v = lane & 1 ? (got | (uint32_t)lo << 16) : ((uint32_t)hi | got << 16);
    const int c = upper * 64 + (lane & ~1);
    st_agent((uint32_t*)(tile + ((size_t)chunk * R + row) * kBfRow + (c >> 5) * 128 + (lane & 1) * 64 + (c & 31) * 2), v);
}

// The same as 16-bit fixed point, one from each lane: one step of a chunk, with its own scale.
__device__ __forceinline__ void store_qhalf(char* tile, int R, int chunk, int step, int row, float y) {
    const int lane = lane_here();
    char* p = tile + (((size_t)chunk * R + row) * 2 + step) * kQHalf;
    const float am = wave_max(fabsf(y));
    const int x = (int)rintf(y * qtile_inv(am)), l = ((x + 128) & 255) - 128;
    const uint32_t mine = (uint32_t)(((x - l) >> 8) & 255) | (uint32_t)(l & 255) << 16;
    const uint32_t next = lane_xor<1>(mine), two = lane & 1 ? next | mine << 8 : mine | next << 8;   // planes of two lanes, of four
    const uint32_t more = lane_xor<2>(two), a = lane & 2 ? more : two, b = lane & 2 ? two : more;
    if ((lane & 3) < 2)
        st_agent((uint32_t*)(p + (lane & 1) * 64 + (lane & 48) + (lane & 12)), lane & 1 ? a >> 16 | (b & 0xffff0000u) : (a & 0xffffu) | b << 16);
    const int sum = wave_sum(x);
    if (lane == 0) st_agent2((float*)(p + 128), am / kQMax, __int_as_float(sum));
}

// 128 columns of one row of the residual stream: x += add; the row's sum of squares over them; x * gain as the next
// projection's input (the norm's 1 / rms is a factor of the row that the projection applies to its result).
template <bool W4>
__device__ __forceinline__ void residual_row(const LayersArgs& a, int blk, int row, float2 x, float2 gains, bool add, float v0, float v1,
                                             float* ssq, bool norm, char* tile) {
    const int lane = lane_here();
    if (add) {
        float* px = a.x + (size_t)row * a.H + blk * 128 + 2 * lane;
        x.x += v0;
        x.y += v1;
        st_agent2(px, x.x, x.y);
    }
    if (!norm) return;                  // behind the last layer
    const float ss = wave_sum(fmaf(x.x, x.x, x.y * x.y));
    if (lane == 0) st_agent(ssq + blk * kLayersRows + row, ss);
    store_tile128<W4>(tile, a.R, blk, row, x.x * gains.x, x.y * gains.y);
}

// what residual_row needs of a row before the sums are there
struct ResidualIn {
    float2 x, gains;
};
__device__ __forceinline__ ResidualIn residual_in(const LayersArgs& a, int blk, int row, const void* gain) {
    const int c = blk * 128 + 2 * (lane_here());
    ResidualIn r{ld_agent2(a.x + (size_t)row * a.H + c), float2{0.f, 0.f}};
    if (gain) r.gains = float2{gain_at(gain, c), gain_at(gain, c + 1)};
    return r;
}

// this lane's share of a row's sum of squares, and the row's 1 / rms from them
__device__ __forceinline__ float row_squares(const LayersArgs& a, const float* ssq, int row) {
    float s = 0.f;
    for (int i = lane_here(); i < a.H / 128; i += 64) s += ld_agent(ssq + i * kLayersRows + row);
    return s;
}
__device__ __forceinline__ float row_rinv(const LayersArgs& a, float squares) {
    return 1.0f / sqrtf(wave_sum(squares) / (float)a.H + a.eps);
}

struct Shared {
    int cursor;                     // of attention's item list
    int last;                       // this workgroup was the last of a column block to arrive
    int given_up;                   // it has stopped waiting for the others (grid_wait)
};

// ---------------- matrix products ----------------
// A unit: the products of up to 16 rows with a block of CB columns over a part of k.  Each wave takes some columns and a share of
// the unit's k, its weights through a ring of registers, the activations from L2 (nobody else in the workgroup wants the
// same ones, so LDS would be a detour); the waves' partial sums meet in LDS, red[share of k][row][CB + 4].
//
// The first weights of a phase are requested in front of its barrier, except by wave 0, which polls there (loads return in order).
// Requested earlier, behind the products by waves that take no part in what follows them, they cost more than they gained (8B
// shape, 1 / 16 requests bf16, 5 requests 4-bit: 1054 / 1489 / 946 us a step): a phase ends with a chain of small loads and
// stores (slabs, arrivals, the residual stream), and under the weights' traffic each of them takes 3 us instead of 1.
// Arrivals counted by wave instead of by workgroup: 938 / 1329 / 835.  A block's rows finished by all its workgroups, each polling
// for the others, instead of by the last to arrive: 909 / 1275 / 785 against 903 / 1193 / 726, the polls hold up the arrivals.
//
// 4-bit weights: the vector ALU is busiest (widening the codes, scales and zero points of every sum), so high and low planes of eight rows
// share a 16-row operand: half the matrix instructions, loads of activations and sums to scale.  Gate/up is not split along k, its
// blocks are every other strip, the columns of one 64-wide step of the down projection's groups, which has its own scale (finer
// than a scale per group, so nothing is lost): slabs and an arrival less, twice the sums to scale in the down projection.  8 layers
// of the 8B shape, 5 requests: 726 -> 678 us (a layer's gate/up 20.7 -> 15.5, down 10.6 -> 10.0).
template <bool W4>
struct Ring {
    static constexpr int PD = 4, NS = W4 ? 4 : 8;   // steps and 16-column strips
    u32x4 w[PD][NS];
    uint32_t sz[W4 ? PD : 1][W4 ? NS : 1];
};

// this wave's part of unit u.  ALT: a block is every other strip of 32 columns.
template <bool W4, int CB, bool ALT>
struct Part {
    static constexpr int CW = W4 ? CB / 64 : 1, KW = kWaves / CW, AHEAD = Ring<W4>::PD;
    const char *W, *SZ;             // the same for the whole wave; a lane's part of an address has 32 bits
    uint32_t w_lane, s_lane;
    size_t strip, sz_strip;         // bytes from one 32-column strip to the next
    int a0, a1, blk, cw, kw, s_only;
    __device__ __forceinline__ Part(const MatP& m, int layer, int u, int s_only_) {
        const int lane = lane_here(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n16 = lane & 15, o = lane >> 4;
        const int split = u / m.nblk, steps = m.K / (W4 ? 128 : 32), kch = m.K / 128;
        blk = u % m.nblk;
        cw = wave % CW;
        kw = wave / CW;
        s_only = s_only_;
        const int k0 = steps * split / m.S, n = steps * (split + 1) / m.S - k0;
        a0 = k0 + n * kw / KW;
        a1 = k0 + n * (kw + 1) / KW;
        const int s0 = ALT ? (blk >> 1) * (CB / 16) + (blk & 1) + cw * 4 : blk * (CB / 32) + cw * 2;
        strip = (size_t)kch * (W4 ? 2048 : 8192);
        W = m.w + (size_t)layer * m.w_step + s0 * strip;
        if (ALT) strip *= 2;
        if constexpr (W4) {
            w_lane = ((o & 1) * 64 + (o >> 1) * 32 + n16) * 16;
            s_lane = n16 * 4;
            sz_strip = (size_t)(s_only ? (kch + 1) >> 1 : kch) * 128;
            SZ = m.sz + (size_t)layer * m.sz_step + s0 * sz_strip;
            if (ALT) sz_strip *= 2;
        } else {
            w_lane = (o * 64 + n16) * 16;
        }
    }
    // bf16: a step of 32 along k, lane octet o <-> k = 32 ks + 8 o .. + 7.  4-bit: a 128-wide group.
    template <bool STREAM>
    __device__ __forceinline__ void load(Ring<W4>& r, int slot, int ks) const {
        const char* p = W + (W4 ? (size_t)ks * 2048 : (size_t)(ks >> 2) * 8192 + (ks & 1) * 4096 + ((ks >> 1) & 1) * 512);
#pragma unroll
        for (int s = 0; s < Ring<W4>::NS; ++s) {
            const u32x4* q = (const u32x4*)(p + (size_t)(s >> 1) * strip + (s & 1) * 256 + w_lane);
            if constexpr (STREAM) r.w[slot][s] = load_stream(q);
            else r.w[slot][s] = *q;
            if constexpr (W4)
                r.sz[slot][s] = *(const uint32_t*)(SZ + (size_t)(s >> 1) * sz_strip + (size_t)(s_only ? ks >> 1 : ks) * 128 + (s & 1) * 64 + s_lane);
        }
    }
    template <bool STREAM>
    __device__ __forceinline__ void prefetch(Ring<W4>& r) const {
#pragma unroll
        for (int i = 0; i < AHEAD; ++i)
            if (a0 + i < a1) load<STREAM>(r, i, a0 + i);
    }
};

// Activations of one step.  bf16: a 16-row operand for each plane.  4-bit: eight rows at most, so the operand's rows 0 to 7 are the rows'
// high planes and 8 to 15 their low planes, one for each 64 along k; with it the (scale, sum) pairs of the two rows that a lane finishes
// (HALF: for each 64 along k).
template <bool W4, bool HALF>
struct Acts {
    u32x4 f[2];
    float2 sx[HALF ? 2 : 1][W4 ? 2 : 1];
};

template <bool W4, bool STREAM, int CB, bool ALT, bool HALF>
__device__ __forceinline__ void unit_sums(const Part<W4, CB, ALT>& p, Ring<W4>& ring, const char* A, int R, float* red) {
    constexpr int NS = Ring<W4>::NS, PD = Ring<W4>::PD, PA = PD, LDR = CB + 4;   // activations PA steps ahead
    constexpr int NV = W4 ? 2 : 4, ROW = !W4 ? kBfRow : HALF ? 2 * kQHalf : kQRow;
    const int lane = lane_here(), n16 = lane & 15, o = lane >> 4, a0 = p.a0, a1 = p.a1;
    const uint32_t a_lane = W4 ? min(n16 & 7, R - 1) * ROW + (n16 >> 3) * 64 + o * 16 : min(n16, R - 1) * ROW + o * 16;
    const auto row = [&](int i) { return W4 ? 4 * (o & 1) + 2 * i + (o >> 1) : 4 * o + i; };   // of this lane's i-th sum
    uint32_t x_lane[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) x_lane[i] = min(row(i), R - 1) * ROW + (HALF ? 128 : 256);
    Acts<W4, HALF> ar[PA];
    const auto load_a = [&](int slot, int ks) {
        if constexpr (W4) {
            const char* q = A + (size_t)ks * R * ROW;
#pragma unroll
            for (int m = 0; m < 2; ++m) ar[slot % PA].f[m] = *(const u32x4*)(q + m * (HALF ? kQHalf : 128) + a_lane);
#pragma unroll
            for (int m = 0; m < (HALF ? 2 : 1); ++m)
#pragma unroll
                for (int i = 0; i < 2; ++i) ar[slot % PA].sx[m][i] = *(const float2*)(q + m * kQHalf + x_lane[i]);
        } else {
            const char* q = A + (size_t)(ks >> 2) * R * kBfRow + (ks & 3) * 128 + a_lane;
            ar[slot % PA].f[0] = *(const u32x4*)q;
            ar[slot % PA].f[1] = *(const u32x4*)(q + 64);
        }
    };
    typedef float Sums __attribute__((ext_vector_type(NV)));
    Sums acc[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) acc[s] = Sums(0.f);
    const auto compute = [&](int slot, int ks) {
        if constexpr (W4) {   // the arithmetic of proj_w4_kernel
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                // scale-only layout: this group's half of the dword; the zero point is 8 everywhere
                const uint32_t szg = p.s_only ? (((ring.sz[slot][s] >> (16 * (ks & 1))) & 0xffffu) | 0x48000000u) : ring.sz[slot][s];
                const __half2 h2 = __builtin_bit_cast(__half2, szg);
                const float sc = __low2float(h2);
                const int nzi = -(int)__high2float(h2);
                i32x4 d = {0, 0, 0, 0};   // lanes 0 to 31: sums of the high plane, rows 4 o + r; the others: those rows' of the low plane
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const uint32_t wa = ring.w[slot][s][2 * m], wb = ring.w[slot][s][2 * m + 1];
                    const i32x4 b = {(int)(wa & 0x0F0F0F0Fu), (int)((wa >> 4) & 0x0F0F0F0Fu), (int)(wb & 0x0F0F0F0Fu),
                                     (int)((wb >> 4) & 0x0F0F0F0Fu)};
                    d = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, ar[slot % PA].f[m]), b, d, 0, 0, 0);
                    if (!HALF && m == 0) continue;
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        int hi = d[2 * i], lo = d[2 * i + 1];
                        swap_rows<32>(hi, lo);   // both planes of row 2 i in the lower lanes, of row 2 i + 1 in the upper ones
                        const float2 sx = ar[slot % PA].sx[HALF ? m : 0][i];
                        const int tot = (hi << 8) + lo + __mul24(nzi, __float_as_int(sx.y));
                        acc[s][i] = fmaf((float)tot, sc * sx.x, acc[s][i]);
                    }
                    if (HALF) d = i32x4{0, 0, 0, 0};
                }
            }
        } else {
#pragma unroll
            for (int pl = 0; pl < 2; ++pl)  // hi plane, then lo plane
#pragma unroll
                for (int s = 0; s < NS; ++s)
                    acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ar[slot % PA].f[pl]),
                                                                   __builtin_bit_cast(bf16x8, ring.w[slot][s]), acc[s], 0, 0, 0);
        }
    };
#pragma unroll
    for (int i = 0; i < PA; ++i)
        if (a0 + i < a1) load_a(i, a0 + i);
    __builtin_amdgcn_sched_barrier(0);
    int ks = a0;
    for (; a1 - ks >= 2 * PD; ks += PD) {   // no branch around the loads while the ring is full
#pragma unroll
        for (int i = 0; i < PD; ++i) {
            compute(i, ks + i);
            __builtin_amdgcn_sched_barrier(0);
            p.template load<STREAM>(ring, i, ks + PD + i);
            load_a(i, ks + PA + i);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    for (; ks < a1; ks += PD) {
#pragma unroll
        for (int i = 0; i < PD; ++i)
            if (ks + i < a1) {
                compute(i, ks + i);
                if (ks + PD + i < a1) p.template load<STREAM>(ring, i, ks + PD + i);
                if (ks + PA + i < a1) load_a(i, ks + PA + i);
            }
    }
#pragma unroll
    for (int i = 0; i < NV; ++i)
        if (row(i) < R) {
#pragma unroll
            for (int s = 0; s < NS; ++s) red[(p.kw * 16 + row(i)) * LDR + p.cw * 64 + s * 16 + n16] = acc[s][i];
        }
}

// What happens to a unit's sums, NR rows a wave.  With a split along k the workgroup that is the last of a block to arrive adds the
// slabs up, in their order.
template <int KW, int CB, int NC, int NR, class Col, class Early, class Done>
__device__ __forceinline__ void unit_finish(const LayersArgs& a, const MatP& m, int layer, int u, const float* red, Shared& sh, Col col, Early early,
                                            Done done) {
    constexpr int LDR = CB + 4;
    const int lane = lane_here(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), R = a.R;
    const int blk = u % m.nblk, split = u / m.nblk;
    const bool mine = wave < R;
    int row[NR];                                    // past the last: that one again, not stored
#pragma unroll
    for (int i = 0; i < NR; ++i) row[i] = min(wave + i * kWaves, R - 1);
    decltype(early(0, 0)) in[NR];
    float v[NR][NC];
    if (mine) {
#pragma unroll
        for (int i = 0; i < NR; ++i) in[i] = early(blk, row[i]);
    }
    __syncthreads();
    if (mine) {
#pragma unroll
        for (int i = 0; i < NR; ++i)
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                float t = 0.f;
#pragma unroll
                for (int k = 0; k < KW; ++k) t += red[(k * 16 + row[i]) * LDR + col(lane, c)];
                v[i][c] = t;
            }
    }
    if (m.S > 1) {
        float* sl = a.slab + (size_t)blk * R * CB;
        const size_t step = (size_t)m.nblk * R * CB;
        if (mine) {
#pragma unroll
            for (int i = 0; i < NR; ++i)
                if (wave + i * kWaves < R) {
#pragma unroll
                    for (int c = 0; c < NC; c += 2) st_agent2(sl + split * step + row[i] * CB + lane * NC + c, v[i][c], v[i][c + 1]);
                }
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            const uint32_t before_me = __hip_atomic_fetch_add(m.arrived + blk * kApart, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            sh.last = before_me + 1 == (uint32_t)m.S * (layer + 1);
        }
        __syncthreads();
        asm volatile("" ::: "memory");
        if (!lds_word(&sh.last) || !mine) return;
#pragma unroll
        for (int i = 0; i < NR; ++i)
#pragma unroll
            for (int c = 0; c < NC; ++c) v[i][c] = 0.f;
        for (int s0 = 0; s0 < m.S; s0 += 8) {
            float2 t[NR][8][NC / 2];
#pragma unroll
            for (int i = 0; i < NR; ++i)
#pragma unroll
                for (int s = 0; s < 8; ++s)
#pragma unroll
                    for (int c = 0; c < NC; c += 2) t[i][s][c / 2] = ld_agent2(sl + min(s0 + s, m.S - 1) * step + row[i] * CB + lane * NC + c);
#pragma unroll
            for (int i = 0; i < NR; ++i)
#pragma unroll
                for (int s = 0; s < 8; ++s)
                    if (s0 + s < m.S) {
#pragma unroll
                        for (int c = 0; c < NC; ++c) v[i][c] += c & 1 ? t[i][s][c / 2].y : t[i][s][c / 2].x;
                    }
        }
    }
    if (mine) {
#pragma unroll
        for (int i = 0; i < NR; ++i)
            if (wave + i * kWaves < R) done(blk, row[i], in[i], v[i]);
    }
}

// A phase: all units of one matrix, false where the launch is to be left.  wait() is the barrier in front of it, col(lane, i) names the NC
// columns of the block that a lane finishes, early(blk, row) loads what done(blk, row, early's result, sums) wants beside the sums.
template <bool W4, bool STREAM, int NC, bool ALT, bool HALF, class Wait, class Col, class Early, class Done>
__device__ __forceinline__ bool matrix_phase(const LayersArgs& a, const MatP& m, int layer, const char* A, float* red, Shared& sh, Wait wait, Col col,
                                             Early early, Done done) {
    constexpr int CB = kBlock;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), units = m.nblk * m.S;
    if ((int)blockIdx.x >= units) {
        wait();
        return !__builtin_amdgcn_readfirstlane(lds_word(&sh.given_up));
    }
    for (int u = blockIdx.x; u < units; u += gridDim.x) {
        const Part<W4, CB, ALT> p(m, layer, u, a.s_only);
        Ring<W4> ring;
        if (wave) p.template prefetch<STREAM>(ring);
        if (u == (int)blockIdx.x) wait();
        else __syncthreads();           // the unit before is done with LDS
        if (!wave) p.template prefetch<STREAM>(ring);
        const int gone = lds_word(&sh.given_up);
        unit_sums<W4, STREAM, CB, ALT, HALF>(p, ring, A, a.R, red);
        if (__builtin_amdgcn_readfirstlane(gone)) return false;   // before the first store: others may still read what lies there
        if (W4 || a.R <= kWaves) unit_finish<Part<W4, CB, ALT>::KW, CB, NC, 1>(a, m, layer, u, red, sh, col, early, done);
        else unit_finish<Part<W4, CB, ALT>::KW, CB, NC, kLayersRows / kWaves>(a, m, layer, u, red, sh, col, early, done);
    }
    return true;
}

// ---------------- the other phases ----------------
// One head of one row of the q/k/v projection: bias, head norm, rotation, then q for attention or the new cache entry
// (rope_append_kernel's arithmetic); lane j holds elements j and j + 64.
struct RopeIn {
    float squares, c, sn;
    int page, slot;
};
__device__ __forceinline__ RopeIn rope_in(const LayersArgs& a, int b) {
    const RopeAppend& p = a.rope;
    const int j = lane_here();
    // lengths and page ids are validated on the host under SUN_VALIDATE; clamp so bad input cannot fault
    const int L = min(max(p.seq_lens[b], 0), p.max_pages * kPageTokens - 1);
    const float2 cs = *(const float2*)(p.table + ((size_t)b * 64 + j) * 2);
    return RopeIn{row_squares(a, a.ssq1, b), cs.x, cs.y,
                  min(max(p.page_tables[(size_t)b * p.max_pages + L / kPageTokens], 0), p.n_pages - 1), L % kPageTokens};
}
__device__ __forceinline__ void rope_row(const LayersArgs& a, int layer, int hh, int b, const RopeIn& in, float lo, float hi) {
    const RopeAppend& p = a.rope;
    const LayerPtrs& w = a.lp[layer - a.l0];
    const int j = lane_here(), D = 128, half = 64;
    float* q_out = a.q + (size_t)(layer % a.ring) * a.q_step;
    if (p.has_bias) {
        const void* bias = hh < p.Hq ? w.bq : hh < p.Hq + p.Hkv ? w.bk : w.bv;
        const int h0 = (hh < p.Hq ? hh : hh < p.Hq + p.Hkv ? hh - p.Hq : hh - p.Hq - p.Hkv) * D;
        lo += gain_at(bias, h0 + j);
        hi += gain_at(bias, h0 + j + half);
    }
    if (p.has_norm && hh < p.Hq + p.Hkv) {
        const float ss = wave_sum(lo * lo + hi * hi);
        const float r = 1.0f / sqrtf(ss / (float)D + a.eps);
        const void* g = hh < p.Hq ? w.qn : w.kn;
        lo = lo * r * gain_at(g, j);
        hi = hi * r * gain_at(g, j + half);
    }
    if (hh < p.Hq + p.Hkv) {
        const float rl = lo * in.c - hi * in.sn, rh = hi * in.c + lo * in.sn;
        lo = rl;
        hi = rh;
    }
    if (hh < p.Hq) {
        st_agent(q_out + ((size_t)b * p.Hq + hh) * D + j, lo);
        st_agent(q_out + ((size_t)b * p.Hq + hh) * D + j + half, hi);
        return;
    }
    if (hh < p.Hq + p.Hkv) {
        uint16_t* kd = p.pool + p.k_base + layer * p.k_layer + (int64_t)in.page * p.k_page + (int64_t)(hh - p.Hq) * p.k_head + in.slot * p.k_token;
        st_agent(kd + j * p.k_dim, f32_to_bf16_bits(lo));
        st_agent(kd + (j + half) * p.k_dim, f32_to_bf16_bits(hi));
    } else {
        uint16_t* vd = p.pool + p.v_base + layer * p.v_layer + (int64_t)in.page * p.v_page + (int64_t)(hh - p.Hq - p.Hkv) * p.v_head + in.slot * p.v_token;
        st_agent(vd + j * p.v_dim, f32_to_bf16_bits(lo));
        st_agent(vd + (j + half) * p.v_dim, f32_to_bf16_bits(hi));
    }
}

// A wave merges the n chunks of one head of one row, c0 the first; the order of the sums is attn_combine_kernel's.  Lane: dims
// 2 lane and 2 lane + 1.
template <bool W4>
__device__ __forceinline__ void merge_row(const AttnArgs& a, int b, int h, int c0, int n, int R, char* tile) {
    constexpr int D = 128, B = 16;            // partial outputs in flight
    const int lane = lane_here();
    const size_t stride = (size_t)a.Hq * (D + 2);
    const float* p = a.partial + (size_t)c0 * stride + (size_t)h * (D + 2);
    float M = -INFINITY, n0 = 0.f, n1 = 0.f, den = 0.f;
    for (int cb = 0; cb < n; cb += 64) {
        const int c = cb + lane, cnt = min(n - cb, 64);
        const float* pj = p + (size_t)cb * stride + 2 * lane;
        const float2 ml = ld_agent2(p + (size_t)min(c, n - 1) * stride + D);
        float2 ov[B];
#pragma unroll
        for (int i = 0; i < B; ++i) ov[i] = ld_agent2(pj + (size_t)min(i, cnt - 1) * stride);
        const float m = c < n ? ml.x : -INFINITY, l = c < n ? ml.y : 0.f;
        float prev;                           // maximum up to the start and to the end of the lane's eight
        const float top = wave_octet_max(m, M, prev);
        const float w = c < n ? exp2f(m - top) : 0.f, sc = exp2f(prev - top);
        M = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(top), 63));
        for (int k0 = 0; k0 < cnt; k0 += B) {
            if (k0) {
#pragma unroll
                for (int i = 0; i < B; ++i) ov[i] = ld_agent2(pj + (size_t)min(k0 + i, cnt - 1) * stride);
            }
#pragma unroll
            for (int i = 0; i < B; ++i)
                if (k0 + i < cnt) {
                    if (i % 8 == 0) {
                        const float s = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(sc), k0 + i));
                        n0 *= s;
                        n1 *= s;
                        den *= s;
                    }
                    const float wk = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w), k0 + i));
                    den = fmaf(wk, __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(l), k0 + i)), den);
                    n0 = fmaf(wk, ov[i].x, n0);
                    n1 = fmaf(wk, ov[i].y, n1);
                }
        }
    }
    store_tile128<W4>(tile, R, h, b, n0 / den, n1 / den);
}

__device__ __forceinline__ const LayersArgs& args_here() { return kernel_args<LayersArgs>(); }

template <bool W4, bool STREAM>
__global__ __launch_bounds__(kWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void layers_kernel(LayersArgs) {
    __shared__ float red[kWaves * 16 * 132];
    __shared__ Shared sh;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (threadIdx.x == 0) sh.given_up = 0;
    __syncthreads();
    uint32_t times;
    const auto arrive = [&]() {
        grid_arrive(args_here().counters, &sh.given_up);
        ++times;
    };
    const auto wait_for = [&](bool fresh) {
        const LayersArgs& a = args_here();
        grid_wait(a.counters, a.lost, times, a.polls, &sh.given_up, fresh);
    };
    const auto wait = [&]() { wait_for(false); };
    int l, l1;
    {
        const LayersArgs& a = args_here();
        l = a.l0;
        l1 = a.l1;
        times = (uint32_t)l * 6 + (l > 0);
        if (l == 0) {
            for (int u = blockIdx.x + gridDim.x * wave; u < a.H / 128 * a.R; u += gridDim.x * kWaves) {
                const ResidualIn in = residual_in(a, u / a.R, u % a.R, a.lp[0].g1);
                residual_row<W4>(a, u / a.R, u % a.R, in.x, in.gains, false, 0.f, 0.f, a.ssq1, true, a.t1);
            }
            arrive();
        }
    }
    const auto pair = [](int lane, int c) { return 2 * lane + c; };
    for (; l < l1; ++l) {
        {   // q/k/v: a block is one head
            const LayersArgs& a = args_here();
            const bool again = l >= a.ring && l % a.ring == 0;   // the tiles of the last `ring` layers are written a second time
            const auto wait_fresh = [&]() { wait_for(again); };
            if (!matrix_phase<W4, STREAM, 2, false, false>(a, a.qkv, l, a.t1 + (size_t)(l % a.ring) * a.h_step, red, sh, wait_fresh, [](int lane, int c) { return lane + 64 * c; },
                                             [&](int, int row) { return rope_in(args_here(), row); },
                                             [&](int blk, int row, const RopeIn& in, const float (&v)[2]) {
                                                 const LayersArgs& b = args_here();
                                                 const float ri = row_rinv(b, in.squares);
                                                 rope_row(b, l, blk, row, in, v[0] * ri, v[1] * ri);
                                             }))
                break;
        }
        arrive();
        {
            const LayersArgs& a = args_here();
            AttnArgs at = a.attn;
            at.kbase += l * a.rope.k_layer;
            at.vbase += l * a.rope.v_layer;
            at.q = a.q + (size_t)(l % a.ring) * a.q_step;
            // with 4-bit weights what depends on the lane does not fit beside the other phases' registers from layer to layer (741 -> 731 us
            // at five requests; the bf16 kernel has the room and would lose 0.3 %)
            attn_split_items<128, 0, true, K_STREAMED>(at, blockIdx.x, gridDim.x, W4 ? lane_here() : threadIdx.x & 63, &sh.cursor, wait);
        }
        arrive();
        {
            const LayersArgs& a = args_here();
            const int Hq = a.attn.Hq, first = blockIdx.x + gridDim.x * wave, total = a.R * Hq;
            int b = min(first, total - 1) / Hq, c0 = a.attn.chunk_off[b], n = a.attn.chunk_off[b + 1] - c0;
            wait();
            for (int u = first; u < total; u += gridDim.x * kWaves) {
                if (u != first) {
                    b = u / Hq;
                    c0 = a.attn.chunk_off[b];
                    n = a.attn.chunk_off[b + 1] - c0;
                }
                merge_row<W4>(a.attn, b, u % Hq, c0, n, a.R, a.ta + (size_t)(l % a.ring) * a.a_step);
            }
        }
        arrive();
        {
            const LayersArgs& a = args_here();
            if (!matrix_phase<W4, STREAM, 2, false, false>(a, a.o, l, a.ta + (size_t)(l % a.ring) * a.a_step, red, sh, wait, pair,
                                             [&](int blk, int row) {
                                                 const LayersArgs& b = args_here();
                                                 return residual_in(b, blk, row, b.lp[l - b.l0].g2);
                                             },
                                             [&](int blk, int row, const ResidualIn& in, const float (&v)[2]) {
                                                 const LayersArgs& b = args_here();
                                                 residual_row<W4>(b, blk, row, in.x, in.gains, true, v[0], v[1], b.ssq2, true, b.t2 + (size_t)(l % b.ring) * b.h_step);
                                             }))
                break;
        }
        arrive();
        {
            const LayersArgs& a = args_here();
            // A block: 64 gate and 64 up columns, 16 and 16 in turn; with 4-bit weights those of one step of the down projection's groups
            if (!matrix_phase<W4, STREAM, 2, W4, false>(a, a.gu, l, a.t2 + (size_t)(l % a.ring) * a.h_step, red, sh, wait,
                                                        [](int lane, int c) { return (lane >> 4) * 32 + (lane & 15) + c * 16; },
                                                        [&](int, int row) {
                                                            const LayersArgs& b = args_here();
                                                            return row_squares(b, b.ssq2, row);
                                                        },
                                                        [&](int blk, int row, float squares, const float (&v)[2]) {
                                                            const LayersArgs& b = args_here();
                                                            const float ri = row_rinv(b, squares), g = v[0] * ri, y = g / (1.f + __expf(-g)) * (v[1] * ri);
                                                            char* t = b.tu + (size_t)(l % b.ring) * b.u_step;
                                                            if constexpr (W4) store_qhalf(t, b.R, blk >> 1, blk & 1, row, y);
                                                            else store_tile64(t, b.R, blk >> 1, blk & 1, row, y);
                                                        }))
                break;
        }
        arrive();
        {
            const LayersArgs& a = args_here();
            if (!matrix_phase<W4, STREAM, 2, false, W4>(a, a.down, l, a.tu + (size_t)(l % a.ring) * a.u_step, red, sh, wait, pair,
                                             [&](int blk, int row) {
                                                 const LayersArgs& b = args_here();
                                                 return residual_in(b, blk, row, l + 1 == b.n_layers ? nullptr : l + 1 < b.l1 ? b.lp[l + 1 - b.l0].g1 : b.g1_next);
                                             },
                                             [&](int blk, int row, const ResidualIn& in, const float (&v)[2]) {
                                                 const LayersArgs& b = args_here();
                                                 residual_row<W4>(b, blk, row, in.x, in.gains, true, v[0], v[1], b.ssq1, l + 1 < b.n_layers, b.t1 + (size_t)((l + 1) % b.ring) * b.h_step);
                                             }))
                break;
        }
        arrive();
    }
    // Where a wait was given up the workgroup has left in the phase behind it, or, from attention's and the merge's, in the o projection, and
    // nobody passes the wait behind that one.  So all that it can have spoilt are partials and tiles of its own items, which at
    // most the merge and the o projection of this layer read: never a cache entry, which comes out of q/k/v.  x is left as
    // it is, others may still read it; the next launch makes not-a-numbers of it.
}

// ---------------- host side ----------------
static size_t up256(size_t v) { return (v + 255) / 256 * 256; }

// Column blocks and split along k.  As many units as there are workgroups at most; every wave that shares k gets a step.
// A row's sums depend on the matrix alone.  Widths whose blocks fill the chip badly lose part of the gain, not all of it (4 layers, launch
// per operation -> this, us): 296 gate/up blocks on 256 workgroups (hidden 3584, ffn 18 944) at 1 / 16 requests 577 -> 489 / 593 -> 591;
// 272 of 4-bit weights (hidden 5120, ffn 17 408) at 1 / 8 406 -> 356 / 415 -> 416, on requests of 2000 to 6000 tokens 422 -> 370 / 508 -> 509 (136 of twice the
// columns, with an operand for each plane: 379 / 435, 398 / 524), bf16 at 1 / 16 724 -> 644 / 747 -> 746; 14B shape 847 ->
// 697 / 886 -> 780, 4-bit 613 -> 554 / 634 -> 600; hidden 8192, ffn 28 672 1351 -> 1258 / 1376 -> 1346, 4-bit 706 -> 607 / 740 -> 655.
static void cut(MatP& m, int N, int K, bool w4) {
    m.K = K;
    m.nblk = N / kBlock;
    m.S = max(1, min(kUnits / m.nblk, w4 ? K / (128 * (kWaves / (kBlock / 64))) : K / (32 * kWaves)));
}

static size_t n_counters(const sun_model_cfg& c) {
    return kCounters * 32 + kApart * (c.n_q_heads + 2 * c.n_kv_heads + 2 * (c.hidden / 128) + c.ffn / 64);
}

struct LayersLayout {
    size_t ssq1, ssq2, slab, t1, ta, t2, tu, q;
    size_t h_step, a_step, u_step, q_step;   // bytes of a layer
    int ring;                                // layers that have tiles of their own
};
// The counters first; ring 0: no room for even one layer.
static LayersLayout layers_layout(const sun_model_cfg& c, int rows, bool w4, size_t bytes) {
    LayersLayout L{};
    const size_t QD = (size_t)c.n_q_heads * c.head_dim, row = w4 ? kQRow : kBfRow;
    size_t off = up256(n_counters(c) * 4);
    const auto take = [&](size_t n) {
        const size_t at = off;
        off += up256(n);
        return at;
    };
    L.ssq1 = take((size_t)c.hidden / 128 * kLayersRows * 4);
    L.ssq2 = take((size_t)c.hidden / 128 * kLayersRows * 4);
    const int Ns[4] = {(c.n_q_heads + 2 * c.n_kv_heads) * 128, c.hidden, 2 * c.ffn, c.hidden}, Ks[4] = {c.hidden, (int)QD, c.hidden, c.ffn};
    size_t slab = 0;
    for (int i = 0; i < 4; ++i) {
        MatP m{};
        cut(m, Ns[i], Ks[i], w4);
        if (m.S > 1) slab = max(slab, (size_t)m.S * rows * Ns[i] * 4);
    }
    L.slab = take(slab);
    L.h_step = up256((size_t)c.hidden / 128 * rows * row);
    L.a_step = up256(QD / 128 * rows * row);
    L.u_step = up256((size_t)c.ffn / 128 * rows * (w4 ? 2 * kQHalf : kBfRow));
    L.q_step = up256(QD * rows * 4);
    const size_t layer = 2 * L.h_step + L.a_step + L.u_step + L.q_step;
    L.ring = (int)min((size_t)c.n_layers, bytes > off ? (bytes - off) / layer : 0);
    L.t1 = take(L.h_step * L.ring);
    L.ta = take(L.a_step * L.ring);
    L.t2 = take(L.h_step * L.ring);
    L.tu = take(L.u_step * L.ring);
    L.q = take(L.q_step * L.ring);
    return L;
}

// The cooperative launch costs about 28 us more than it saves outside the layers, and a layer saves, at the narrowest widths that were
// timed (hidden 1024; wider ones two or three times that), 17 us at one row down to 7 at 16 (bf16), 13 at one row down to 10 at 8
// (4-bit): few layers are faster with a launch per operation.  Hidden 1024, launch per operation -> this (us), at 1 / 12 / 16 rows: one layer 65 / 72 / 71 ->
// 77 / 89 / 92, two 112 / 123 / 127 -> 107 / 134 / 141, three 158 / 174 / 177 -> 135 / 173 / 187, four 212 / 226 / 235 -> 174 / 215 / 241, six 303 / 334 / 343 ->
// 234 / 302 / 335, eight 415 / 451 / 471 -> 307 / 402 / 441; 4-bit at 1 / 8 rows, one layer 59 / 65 -> 75 / 84, two 100 / 111 -> 103 / 119, three 141 / 157 ->
// 133 / 154, four 188 / 200 -> 161 / 188, six 264 / 293 -> 217 / 262.  The line keeps clear of what is slower: it was drawn when a layer saved 4 us
// at 16 rows and at 8 of 4-bit weights, and sends stacks to separate launches that break even or better here today: at 16 rows five and six layers (288 ->
// 288, 343 -> 335; hidden 2048 from two on, 179 -> 177, six 470 -> 398), 4-bit at 8 three to six (hidden 2048 three 186 -> 170, six 347 -> 289).
static bool layers_shape(const Weights& W, int rows) {
    return W.cfg.act_dtype == SUN_BF16 && W.cfg.head_dim == 128 && rows <= (W.quant ? kLayersRowsW4 : kLayersRows) &&
           W.cfg.n_layers * ((W.quant ? 12 : 20) - rows) >= 26;
}

int resident_grid(const void* kernel, int threads, int most, int dev) {
    int coop = 0, cus = 0, per = 0;
    const bool ok = hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) == hipSuccess && coop &&
                    hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
                    hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, threads, 0) == hipSuccess && per >= 1;
    return ok ? min(cus, most) : 0;
}

bool is_capturing(hipStream_t st) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    return hipStreamIsCapturing(st, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone;
}

// Whether a stream's work may run on all compute units: a workgroup that needs a unit which its stream may not use never comes.
bool has_all_units(hipStream_t st) {
    int dev = 0, cus = 0;
    uint32_t mask[32] = {};                               // 0.5 us a call
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus > 32 * 32) return false;
    if (hipExtStreamGetCUMask(st, (cus + 31) / 32, mask) != hipSuccess) return false;
    for (int i = 0; i < cus; ++i)
        if (!(mask[i / 32] >> (i % 32) & 1)) return false;
    return true;
}

constexpr int kVariants = 3;
static int layers_variant(const Weights& W) { return W.quant ? 2 : W.layers[0].qkv.stream; }
static const void* layers_fn(int variant) {
    return variant == 2 ? (const void*)layers_kernel<true, false> : variant == 1 ? (const void*)layers_kernel<false, true> : (const void*)layers_kernel<false, false>;
}

static int layers_grid(int variant) {
    constexpr int kDevices = 64;
    static std::atomic<int> known[kVariants][kDevices];   // grid + 1 of a kernel on a device
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevices) return 0;
    int g = known[variant][dev].load(std::memory_order_relaxed);
    if (g == 0) {
        g = resident_grid(layers_fn(variant), kWaves * 64, kUnits, dev) + 1;
        known[variant][dev].store(g, std::memory_order_relaxed);
    }
    return g - 1;
}

bool layers_usable(const Weights& W, int rows, const LayersScratch& scratch, hipStream_t st) {
    if (!layers_shape(W, rows) || layers_layout(W.cfg, rows, W.quant, scratch.bytes).ring < 1 || is_capturing(st)) return false;
    return has_all_units(st) && layers_grid(layers_variant(W)) > 0;
}

LayersZero layers_zero(const LayersScratch& scratch, const Weights& W, const AttnPlan& plan) {
    return LayersZero{(uint32_t*)scratch.p, (int)n_counters(W.cfg), layers_lost(plan)};
}

hipError_t launch_layers(const KvPool& pool, const Weights& W, int rows, float* x, const float* table, const AttnPlan& plan,
                         const int32_t* page_tables, int max_pages, const int32_t* seq_lens, int total_chunks_hint, int full_chunks_hint,
                         const LayersScratch& scratch, unsigned polls, hipStream_t st) {
    const sun_model_cfg& c = W.cfg;
    const sun_kv_layout& P = pool.lay;
    const LayersLayout L = layers_layout(c, rows, W.quant, scratch.bytes);
    if (!layers_shape(W, rows) || L.ring < 1 || P.k_dim != 1 || P.k_token != 128 || P.v_token != 1 || P.v_dim != kPageTokens) return hipErrorInvalidValue;
    char* base = (char*)scratch.p;
    const bool w4 = W.quant;
    LayersArgs a{};
    uint32_t* arrived = (uint32_t*)base + kCounters * 32;
    const auto mat = [&](const Mat LayerW::*which) {
        const Mat &m0 = W.layers[0].*which, &m1 = W.layers[c.n_layers > 1 ? 1 : 0].*which;
        MatP m{};
        m.w = (const char*)m0.w;
        m.w_step = (const char*)m1.w - (const char*)m0.w;   // the packed layers lie one like the other
        m.sz = (const char*)m0.sz;
        m.sz_step = w4 ? (const char*)m1.sz - (const char*)m0.sz : 0;
        cut(m, m0.N, m0.K, w4);
        m.arrived = arrived;
        arrived += m.nblk * kApart;
        return m;
    };
    a.qkv = mat(&LayerW::qkv);
    a.o = mat(&LayerW::o);
    a.gu = mat(&LayerW::gu);
    a.down = mat(&LayerW::down);
    a.attn = make_attn_args(pool, 0, plan, nullptr, page_tables, max_pages, seq_lens, 1, rows);
    if (total_chunks_hint >= 0 && full_chunks_hint >= 0) {
        a.attn.n_full_items = full_chunks_hint * c.n_kv_heads;
        a.attn.total_items = total_chunks_hint * c.n_kv_heads;
    }
    a.rope = RopeAppend{table, seq_lens, page_tables, pool.base, P.k_off, P.k_layer, P.k_page, P.k_head, P.k_token, P.k_dim,
                        P.v_off, P.v_layer, P.v_page, P.v_head, P.v_token, P.v_dim, c.n_q_heads, c.n_kv_heads, max_pages, (int)P.n_pages,
                        c.qk_norm, c.qkv_bias};
    a.x = x;
    a.ssq1 = (float*)(base + L.ssq1);
    a.ssq2 = (float*)(base + L.ssq2);
    a.slab = (float*)(base + L.slab);
    a.counters = (uint32_t*)base;
    a.lost = layers_lost(plan);
    a.polls = polls;
    a.ring = L.ring;
    a.t1 = base + L.t1;
    a.ta = base + L.ta;
    a.t2 = base + L.t2;
    a.tu = base + L.tu;
    a.q = (float*)(base + L.q);
    a.h_step = L.h_step;
    a.a_step = L.a_step;
    a.u_step = L.u_step;
    a.q_step = L.q_step / 4;
    a.n_layers = c.n_layers;
    a.R = rows;
    a.H = c.hidden;
    a.s_only = w4 && W.layers[0].qkv.s_only;
    a.eps = c.rms_eps;
    const void* fn = layers_fn(layers_variant(W));
    const int grid = layers_grid(layers_variant(W));
    if (grid < 1) return hipErrorNotSupported;
    for (int l0 = 0; l0 < c.n_layers; l0 += kLayersPerLaunch) {
        a.l0 = l0;
        a.l1 = min(c.n_layers, l0 + kLayersPerLaunch);
        for (int l = l0; l < a.l1; ++l) {
            const LayerW& w = W.layers[l];
            a.lp[l - l0] = LayerPtrs{w.g1, w.g2, w.qn, w.kn, w.bq, w.bk, w.bv};
        }
        a.g1_next = a.l1 < c.n_layers ? W.layers[a.l1].g1 : nullptr;
        void* args[] = {&a};
        if (hipError_t e = hipLaunchCooperativeKernel(fn, dim3(grid), dim3(kWaves * 64), args, 0, st)) return e;
    }
    return hipSuccess;
}

}  // namespace sun
