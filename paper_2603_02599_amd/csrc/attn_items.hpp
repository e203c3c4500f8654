// The cache-reading part of a decode step's attention (bf16), shared by the launch of its own (attention.hip) and by the launch
// that runs all layers of a small batch (layers.hip).
#pragma once
#include <type_traits>

#include "kernels.hpp"

namespace sun {

constexpr int CH = kAttnChunk;
constexpr float kLog2e = 1.4426950408889634f;
constexpr int kRecInts = 24;  // ints per item record
constexpr int kTopUp = CH / kAttnSmall;  // small chunks that stand for one full chunk in a wave's item list

struct AttnArgs {
    const uint16_t* kbase;  // pool base + k_off + layer * k_layer
    const uint16_t* vbase;
    int64_t k_page, k_head, v_page, v_head;
    const float* q;         // [batch, Hq*D]
    const int32_t* page_tables;
    const int32_t* n_or_len;
    const int32_t* chunk_off;
    const int32_t* full_off;
    const int32_t* records;
    float* partial;
    int len_plus, max_pages, batch, Hq, Hkv, n_pages;
    int n_full_items, total_items;  // item counts when the host knows the lengths, else -1: read from the plan
    float qscale;           // log2(e) / sqrt(D)
};

inline AttnArgs make_attn_args(const KvPool& pool, int layer, const AttnPlan& plan, const float* q, const int32_t* page_tables, int max_pages,
                               const int32_t* n_or_len, int len_plus, int batch) {
    const sun_model_cfg& c = pool.cfg;
    const sun_kv_layout& L = pool.lay;
    AttnArgs a{};
    a.kbase = pool.base + L.k_off + (int64_t)layer * L.k_layer;
    a.vbase = pool.base + L.v_off + (int64_t)layer * L.v_layer;
    a.k_page = L.k_page;
    a.k_head = L.k_head;
    a.v_page = L.v_page;
    a.v_head = L.v_head;
    a.q = q;
    a.page_tables = page_tables;
    a.n_or_len = n_or_len;
    a.chunk_off = plan.chunk_off;
    a.full_off = plan.full_off;
    a.records = plan.records;
    a.partial = plan.partial;
    a.len_plus = len_plus;
    a.max_pages = max_pages;
    a.batch = batch;
    a.Hq = c.n_q_heads;
    a.Hkv = c.n_kv_heads;
    a.n_pages = (int)L.n_pages;
    a.qscale = kLog2e / sqrtf((float)c.head_dim);
    a.n_full_items = a.total_items = -1;
    return a;
}

// hi and lo bf16 of two fp32 values
__device__ __forceinline__ void split_pair(float x0, float x1, uint32_t& hi, uint32_t& lo) {
    hi = pack_bf16(x0, x1);
    lo = pack_bf16(x0 - bf16_lo(hi), x1 - bf16_hi(hi));
}

// The items of workgroup wg out of nwg, by its eight waves.  GT: query heads per KV head, 0: taken from the arguments; eight at most
// (kMaxGroup, which every model is checked for): rows 8 to 15 of the operand of heads are nobody's and are not stored.
// SHARED: the partials are read again by other workgroups of the same launch.  list_cursor: LDS; the previous use of it is over.
// before() (SHARED) is what to wait for before q and the newest entry of every request may be read; items without the newest
// entry request their first K and V in front of it, except for wave 0's, which polls there.
template <int D, int GT, bool SHARED, KRead K_READ, class Before>
__device__ __forceinline__ void attn_split_items(const AttnArgs& a, int wg, int nwg, int lane, int* list_cursor, Before before) {
    const int G = GT ? GT : a.Hq / a.Hkv;
    constexpr int NS = D / 32;  // dim slices of a QK MFMA
    constexpr int NB = D / 16;  // dim blocks of a PV MFMA
    static_assert(GT <= kMaxGroup && kMaxGroup <= 8 && NB % 4 == 0, "partials of eight heads leave in stores of four blocks");
    constexpr bool QUADS = NS == 4;  // operand register s holds dims 32 kq + 8 s instead of 32 s + 8 kq
    constexpr bool ROWS = K_READ != K_IN_PLACE;  // K in whole token rows and through turn_k
    static_assert(QUADS || !ROWS, "a row of 64 dims is not four quads'");
    const int c16 = lane & 15, kq = lane >> 4;
    // One workgroup of 8 waves per compute unit.  Items are dealt to workgroups statically: full
    // chunks (all of one size) round-robin; the workgroups that got one full chunk fewer are
    // topped up with a block of kTopUp small chunks, the remaining small chunks go round-robin.
    // Inside a workgroup the waves take the list's entries in order through a counter in LDS, so
    // they run out of work within one small chunk of each other however unevenly the hardware
    // serves them.  Which wave computes an item has no effect on its value.
    if (threadIdx.x == 0) *list_cursor = 0;
    __syncthreads();
    const int n_full = a.n_full_items >= 0 ? a.n_full_items : a.full_off[a.batch] * a.Hkv;
    const int total_items = a.total_items >= 0 ? a.total_items : a.chunk_off[a.batch] * a.Hkv;
    const int n_small = total_items - n_full;
    const int fq = n_full / nwg, fr = n_full % nwg;
    auto next_item = [&]() -> int {  // next unclaimed entry of this workgroup's list, total_items when it is over
        int c = 0;
        if (lane == 0) c = atomicAdd(list_cursor, 1);
        c = __builtin_amdgcn_readfirstlane(c);
        const int mine_full = fq + (wg < fr ? 1 : 0);
        if (c < mine_full) return wg + c * nwg;
        c -= mine_full;
        const int top = wg >= fr ? min(max(n_small - kTopUp * (wg - fr), 0), kTopUp) : 0;
        if (c < top) return n_full + kTopUp * (wg - fr) + c;
        c -= top;
        const long long j = (long long)kTopUp * (nwg - fr) + wg + (long long)c * nwg;
        return j < n_small ? n_full + (int)j : total_items;
    };

    const auto put = [](float* p, float v) {
        if constexpr (SHARED) st_agent(p, v);
        else *p = v;
    };
    // K operand rows: MFMA row i of tile 0 <-> page (i>>3), token 8*((i>>2)&1) + (i&3); tile 1: +4
    const int k_psel = c16 >> 3, k_tok = 8 * ((c16 >> 2) & 1) + (c16 & 3);
    constexpr int SLICE = QUADS ? 8 : 32, OCTET = QUADS ? 32 : 8;   // dims from one register, from one kq to the next
    const int64_t k_lane_off = (int64_t)k_tok * D + kq * OCTET;
    // V^T operand: lane (dim c16 of a 16-dim block, token octet kq): page (kq>>1), tokens 8*(kq&1)..+7
    const int v_psel = kq >> 1;
    const int64_t v_lane_off = (int64_t)c16 * kPageTokens + 8 * (kq & 1);

    auto load_rec = [&](int it) { return lane < kRecInts ? a.records[(size_t)it * kRecInts + lane] : 0; };
    u32x4_s kr[2][NS], vr[NB];  // K and V^T operand registers of one 32-token page pair
    auto load_k = [&](int recv, int head, int pp) {
        const int pA = __builtin_amdgcn_readlane(recv, 2 * pp);
        int pB = __builtin_amdgcn_readlane(recv, 2 * pp + 1);
        if (pB < 0) pB = pA;
        const uint16_t* kh = a.kbase + head * a.k_head;
        if constexpr (ROWS) {
            const uint16_t* kp = kh + (int64_t)(lane & 8 ? pB : pA) * a.k_page + ((lane >> 2) & 1) * 8 * D + kq * 32 + (lane & 3) * 8;
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const u32x4_s* row = reinterpret_cast<const u32x4_s*>(kp + (4 * t + r) * D);
                    kr[t][r] = K_READ == K_STREAMED ? load_stream(row) : *row;
                }
            return;
        }
        const uint16_t* kp = kh + (int64_t)(k_psel ? pB : pA) * a.k_page + k_lane_off;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            kr[0][s] = *reinterpret_cast<const u32x4_s*>(kp + s * SLICE);
            kr[1][s] = *reinterpret_cast<const u32x4_s*>(kp + 4 * D + s * SLICE);
        }
    };
    // V^T is requested with streaming loads: every instruction reads two runs of 512 contiguous bytes, which
    // such loads move 10 % faster than cached ones and without displacing what the neighbouring kernels exchange
    // through the caches.  On half cache lines they are slower than cached ones (a read-only kernel: 6.7 against 6.1 TB/s on
    // contiguous kilobytes, 5.95 against 6.2 on 64 bytes of each of 16 rows), which is what K's operand is in the cache's layout: lane
    // (token, eight dims).  So K of 128 dims is read in whole token rows instead, four lanes side by side on 64 bytes,
    // register r the tokens 8 half + r (+ 4), and turn_k exchanges register and lane of four: behind it register s holds dims 32 kq + 8 s of the
    // lane's token.  Streamed so, against cached loads of the operand as it lies (us, 8 layers of the 8B shape, one process
    // in turn): 64 requests 2216 -> 2198, 150 (4-bit) 3176 -> 3120, 256 5355 -> 5235, 14B shape with 24 long requests 3352 -> 3357; read so without
    // streaming 2221 / 3174 / 5354 / 3360, the operand as it lies streamed 2275 / 3316 / 5735 / 3509 (2242 / 3269 / 5641 / 3345 beside them).
    auto load_v = [&](int recv, int head, int pp) {
        const int pA = __builtin_amdgcn_readlane(recv, 2 * pp);
        int pB = __builtin_amdgcn_readlane(recv, 2 * pp + 1);
        if (pB < 0) pB = pA;
        const uint16_t* vp = a.vbase + head * a.v_head + (int64_t)(v_psel ? pB : pA) * a.v_page + v_lane_off;
#pragma unroll
        for (int b = 0; b < NB; ++b) vr[b] = load_stream(reinterpret_cast<const u32x4_s*>(vp + b * 16 * kPageTokens));
    };

    auto turn_k = [&]() {
        if constexpr (ROWS) {
            const bool b0 = lane & 1, b1 = lane & 2;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    uint32_t x[4];
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const uint32_t lo = kr[t][j][w], hi = kr[t][j + 2][w], up = lane_xor<2>(hi), down = lane_xor<2>(lo);
                        x[j] = b1 ? up : lo;
                        x[j + 2] = b1 ? hi : down;
                    }
#pragma unroll
                    for (int j = 0; j < 4; j += 2) {
                        const uint32_t up = lane_xor<1>(x[j + 1]), down = lane_xor<1>(x[j]);
                        kr[t][j][w] = b0 ? up : x[j];
                        kr[t][j + 1][w] = b0 ? x[j + 1] : down;
                    }
                }
        }
    };
    bf16x8 qhi[NS], qlo[NS];
    // q as MFMA B operand, hi + lo bf16: lane (head g = c16, dim octet kq) per slice s, the dims of K's registers
    auto load_q = [&](int req, int head) {
        const float* qp = a.q + ((size_t)req * a.Hq + head * G + (c16 < G ? c16 : 0)) * D;
        f32x4 q[NS][2];
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int i = 0; i < 2; ++i) q[s][i] = *reinterpret_cast<const f32x4*>(qp + kq * OCTET + s * SLICE + 4 * i);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            u32x4_s h, l;
#pragma unroll
            for (int p = 0; p < 4; ++p) {   // with the hardware's converter: rounded by hand, a change of item took 0.3 to 0.8 % of a step longer
                uint32_t hi, lo;
                split_pair(c16 < G ? q[s][p >> 1][2 * (p & 1)] * a.qscale : 0.f, c16 < G ? q[s][p >> 1][2 * (p & 1) + 1] * a.qscale : 0.f, hi, lo);
                h[p] = hi;
                l[p] = lo;
            }
            qhi[s] = __builtin_bit_cast(bf16x8, h);
            qlo[s] = __builtin_bit_cast(bf16x8, l);
        }
    };

    // current item state (wave-uniform scalars) and accumulators
    int item = total_items, item_n = total_items, rec = 0;
    const auto claim = [&]() {
        item = next_item();
        if (item >= total_items) return;
        item_n = next_item();
        rec = load_rec(item);
    };
    bool requested = false;
    if (!SHARED || threadIdx.x >= 64) claim();
    if constexpr (SHARED) {
        if (item < total_items && !__builtin_amdgcn_readlane(rec, 21)) {
            load_k(rec, __builtin_amdgcn_readlane(rec, 17), 0);
            load_v(rec, __builtin_amdgcn_readlane(rec, 17), 0);
            requested = true;
        }
        before();
        if (threadIdx.x < 64) claim();
    }
    if (item >= total_items) return;
    int req = __builtin_amdgcn_readlane(rec, 16), head = __builtin_amdgcn_readlane(rec, 17);
    int t0 = __builtin_amdgcn_readlane(rec, 18), t1 = __builtin_amdgcn_readlane(rec, 19);
    int cidx = __builtin_amdgcn_readlane(rec, 20);
    int npairs = ((t1 - t0 + kPageTokens - 1) / kPageTokens + 1) / 2, pp = 0;
    if (!requested) {
        load_k(rec, head, 0);
        load_v(rec, head, 0);
    }
    int rec_n = load_rec(item_n < total_items ? item_n : item);
    load_q(req, head);
    int head_n = __builtin_amdgcn_readlane(rec_n, 17);

    f32x4 O[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) O[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f;

    // One pipeline step = one 32-token page pair.  On entry K of the pair has been requested
    // earlier and V is still in flight.  K of the following pair (of this item or of the wave's
    // next item) is requested as soon as the score MFMAs have consumed the K registers, V of the
    // following pair right after the output MFMAs.  The wave's last pair requests nothing.
    auto step = [&](auto is_last) {
        constexpr bool LAST = decltype(is_last)::value;
        f32x4 sx = {0.f, 0.f, 0.f, 0.f}, sy = {0.f, 0.f, 0.f, 0.f};
        turn_k();
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const bf16x8 kx = __builtin_bit_cast(bf16x8, kr[0][s]), ky = __builtin_bit_cast(bf16x8, kr[1][s]);
            sx = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kx, qhi[s], sx, 0, 0, 0);
            sy = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ky, qhi[s], sy, 0, 0, 0);
            sx = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kx, qlo[s], sx, 0, 0, 0);
            sy = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ky, qlo[s], sy, 0, 0, 0);
        }
        // The following pair is requested unconditionally (branch-free, so that the K and V
        // requests can stay in flight across each other).
        const bool more_pairs = pp + 1 < npairs;
        const int nrec = more_pairs ? rec : rec_n, nhead = more_pairs ? head : head_n, npp = more_pairs ? pp + 1 : 0;
        if constexpr (!LAST) load_k(nrec, nhead, npp);

        // this lane: head c16, tokens tb + r (tile X) and tb + 4 + r (tile Y)
        const int tb = t0 + pp * 32 + (kq >> 1) * 16 + 8 * (kq & 1);
        float mloc = -INFINITY;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            sx[r] = (tb + r < t1) ? sx[r] : -INFINITY;
            sy[r] = (tb + 4 + r < t1) ? sy[r] : -INFINITY;
            mloc = fmaxf(mloc, fmaxf(sx[r], sy[r]));
        }
        mloc = fmaxf(mloc, lane_xor<16>(mloc));
        mloc = fmaxf(mloc, lane_xor<32>(mloc));
        const float m_new = fmaxf(m_run, mloc);
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        m_run = m_new;
        float p[8], psum = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            p[r] = __builtin_amdgcn_exp2f(sx[r] - m_new);
            p[4 + r] = __builtin_amdgcn_exp2f(sy[r] - m_new);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) psum += p[e];
        l_run = l_run * alpha + psum;
        u32x4_s ph, pl;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint32_t hi, lo;
            split_pair(p[2 * e], p[2 * e + 1], hi, lo);
            ph[e] = hi;
            pl[e] = lo;
        }
        const bf16x8 phi = __builtin_bit_cast(bf16x8, ph), plo = __builtin_bit_cast(bf16x8, pl);
        // rescale O only when some head's running maximum moved (rare after the first pairs);
        // row (head) 4*kq + r of the output tile needs alpha of lane (head)
        if (__any(alpha != 1.f)) {
            float al[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) al[r] = __shfl(alpha, 4 * kq + r);
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) O[b][r] *= al[r];
        }
        // pool slots past the end of the cache may hold anything: zero their V
        if (t0 + pp * 32 + 32 > t1) {
            const int vt = t0 + pp * 32 + (kq >> 1) * 16 + 8 * (kq & 1);
            uint32_t msk[4];
#pragma unroll
            for (int w = 0; w < 4; ++w)
                msk[w] = (vt + 2 * w < t1 ? 0x0000ffffu : 0u) | (vt + 2 * w + 1 < t1 ? 0xffff0000u : 0u);
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int w = 0; w < 4; ++w) vr[b][w] &= msk[w];
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const bf16x8 vt8 = __builtin_bit_cast(bf16x8, vr[b]);
            O[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(phi, vt8, O[b], 0, 0, 0);
            O[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(plo, vt8, O[b], 0, 0, 0);
        }
        if constexpr (!LAST) {
            load_v(nrec, nhead, npp);
            if (++pp < npairs) return;
        }

        float l_tot = l_run + lane_xor<16>(l_run);
        l_tot += lane_xor<32>(l_tot);
        float* pbase = a.partial + ((size_t)cidx * a.Hq + head * G) * (D + 2);
        // Rows of 16 lanes hold heads 4 kq + r, 16 dims of each register's block: the first four heads' and the next four's
        // rows of four blocks are exchanged into one register, 64 dims of a head that a wave stores together.
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int b = 0; b < NB; b += 4) {
                float x[4] = {O[b][r], O[b + 1][r], O[b + 2][r], O[b + 3][r]};
                swap_rows<16>(x[0], x[1]);   // rows 0 and 1 of x[0]: head r's of blocks b and b + 1, of x[1]: head 4 + r's
                swap_rows<16>(x[2], x[3]);
                swap_rows<32>(x[0], x[2]);
                swap_rows<32>(x[1], x[3]);
                if (r < G) put(pbase + (size_t)r * (D + 2) + b * 16 + lane, x[0]);
                if (4 + r < G) put(pbase + (size_t)(4 + r) * (D + 2) + b * 16 + lane, x[1]);
            }
        if (kq == 0 && c16 < G) {
            put(pbase + (size_t)c16 * (D + 2) + D, m_run);
            put(pbase + (size_t)c16 * (D + 2) + D + 1, l_tot);
        }
        if constexpr (LAST) return;
        item = item_n;
        item_n = next_item();
        rec = rec_n;
        req = __builtin_amdgcn_readlane(rec, 16);
        head = __builtin_amdgcn_readlane(rec, 17);
        t0 = __builtin_amdgcn_readlane(rec, 18);
        t1 = __builtin_amdgcn_readlane(rec, 19);
        cidx = __builtin_amdgcn_readlane(rec, 20);
        npairs = ((t1 - t0 + kPageTokens - 1) / kPageTokens + 1) / 2;
        pp = 0;
        rec_n = load_rec(item_n < total_items ? item_n : item);
        load_q(req, head);  // also drains every outstanding request before the steady state resumes
        head_n = __builtin_amdgcn_readlane(rec_n, 17);
#pragma unroll
        for (int b = 0; b < NB; ++b) O[b] = f32x4{0.f, 0.f, 0.f, 0.f};
        m_run = -INFINITY;
        l_run = 0.f;
    };

    while (pp + 1 < npairs || item_n < total_items) step(std::false_type{});
    step(std::true_type{});
}

}  // namespace sun
