// Paged GQA decode attention over the shared KV pool (the cache-reading part of
// Eq. 3; the cache is prompt KV from any task's prefill module followed by
// decode-generated KV, Eq. 4).  One query position per request attends to all
// n_i cached positions of that request; requests of different source models are
// handled identically, the pool is addressed through the page table only.
//
// Work decomposition: a work item is (request, kv head, chunk of positions).  All but the last
// 256..511 positions of a request form full chunks of 256, the rest small chunks of 64 (below 64
// requests the full chunks are shorter, see attn_full_chunk); the chunk grid of a request depends on
// its own length and the batch size only, so a request's result does not depend on its batch-mates.  One persistent workgroup of 8 waves per compute unit works through a
// statically dealt item list, full chunks first; a wave streams an item's K and V^T pages with
// 16-byte loads straight into matrix-core operand registers:
//   S^T[token, head] = K[token, :] . q[head, :]      (16x16x32 MFMA, q split hi+lo bf16)
//   O[head, dim]    += P[head, token] V^T[dim, token] (16x16x32 MFMA, P split hi+lo bf16)
// The group's q heads occupy the first G of the 16 MFMA columns.  Softmax runs in
// fp32 in the log2 domain with a running maximum; partial (O, m, l) per item are
// merged by a second kernel in chunk order.  The matrix cores are used because at
// ~13 HBM bytes per CU-clock the vector ALUs cannot also convert, multiply and
// reduce 256 bf16 values per token for several query heads; the kernel stays HBM
// bound.  An fp32 vector-ALU variant serves the fp32 parity configuration.
#include "attn_items.hpp"
#include "kernels.hpp"
#include "rows.hpp"

namespace sun {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

size_t attn_max_chunks(int batch, int max_pages, int Hkv) {
    // An upper bound for every batch size up to `batch` (a workspace sized for a larger batch serves a smaller
    // one).  Full chunks of a request: n / ch with ch = 256, or a shorter ch only while n * Hkv * b / 2048 < 256,
    // which bounds b * n / ch by 4096 / Hkv over the b < 64 requests; small chunks: at most
    // (2 * 256 - 1) / 64 + 1 = 8 per request.
    const size_t max_tokens = (size_t)max_pages * kPageTokens;
    return (size_t)batch * (max_tokens / CH + 2 * CH / kAttnSmall + 1) + 4096 / (size_t)Hkv + 64;
}

// ---------------------------------------------------------------------------------
// plan: chunk counts of every request, their prefix sums, and one record per work item
// ---------------------------------------------------------------------------------
// Items of all full chunks come first, ordered (request, kv head, chunk), then the items of all small chunks in the same
// order.  Record: the chunk's page ids (clamped into the pool, -1 where the chunk has no page), then request, kv head,
// first and one-past-last token, the chunk's slot in the partial array (chunks of a request in token order), and whether it
// holds the request's last token.
// Every workgroup sums up the chunk counts of all requests for itself (at most 1024 of them, four a thread), so that no
// launch has to come first; workgroup 0 stores the prefix sums for the kernels that follow.
struct PlanArgs {
    const int32_t* n_or_len;
    const int32_t* page_tables;
    int32_t *chunk_off, *full_off, *records;
    int len_plus, batch, max_pages, n_pages, Hkv;
};

__device__ __forceinline__ void attn_plan_block(const PlanArgs& a, int block, int n_blocks) {
    __shared__ int f_off[1025], s_off[1025], wave_f[4], wave_s[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, max_tokens = a.max_pages * kPageTokens;
    int nf[4], ns[4], f = 0, sm = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = tid * 4 + i;
        int ch;
        nf[i] = ns[i] = 0;
        if (r < a.batch) attn_chunking(min(max(a.n_or_len[r] + a.len_plus, 1), max_tokens), a.batch, a.Hkv, nf[i], ns[i], ch);
        f += nf[i];
        sm += ns[i];
    }
    int fi = f, si = sm;   // inclusive over the wave, then over the workgroup
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int uf = __shfl_up(fi, o), us = __shfl_up(si, o);
        if (lane >= o) {
            fi += uf;
            si += us;
        }
    }
    if (lane == 63) {
        wave_f[wave] = fi;
        wave_s[wave] = si;
    }
    __syncthreads();
    int bf = fi - f, bs = si - sm;
#pragma unroll
    for (int w = 0; w < 4; ++w)
        if (w < wave) {
            bf += wave_f[w];
            bs += wave_s[w];
        }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = tid * 4 + i;
        if (r <= a.batch) {
            f_off[r] = bf;
            s_off[r] = bs;
        }
        bf += nf[i];
        bs += ns[i];
    }
    if (tid == 255 && a.batch == 1024) {
        f_off[1024] = bf;
        s_off[1024] = bs;
    }
    __syncthreads();
    if (block == 0)
        for (int r = tid; r <= a.batch; r += 256) {
            a.full_off[r] = f_off[r];
            a.chunk_off[r] = f_off[r] + s_off[r];
        }
    const int total_full = f_off[a.batch] * a.Hkv, total = total_full + s_off[a.batch] * a.Hkv;
    for (int item = block * 16 + (tid >> 4); item < total; item += n_blocks * 16) {
        const int slot = tid & 15;
        const bool is_full = item < total_full;
        const int* off = is_full ? f_off : s_off;
        const int idx = is_full ? item : item - total_full;
        int lo = 0, hi = a.batch;  // request whose item range [off[r]*Hkv, off[r+1]*Hkv) holds idx
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (off[mid] * a.Hkv <= idx) lo = mid; else hi = mid;
        }
        const int req = lo, nc = off[req + 1] - off[req];
        const int local = idx - off[req] * a.Hkv, head = local / nc, cj = local % nc;
        const int n = min(max(a.n_or_len[req] + a.len_plus, 1), max_tokens);
        const int nfull = f_off[req + 1] - f_off[req];
        const int ch = attn_full_chunk(n, a.batch, a.Hkv);
        const int t0 = is_full ? cj * ch : nfull * ch + cj * kAttnSmall;
        const int t1 = is_full ? t0 + ch : min(n, t0 + kAttnSmall);
        const int npages = (t1 - t0 + kPageTokens - 1) / kPageTokens;
        int32_t* rec = a.records + (size_t)item * kRecInts;
        rec[slot] = slot < npages ? min(max(a.page_tables[(size_t)req * a.max_pages + t0 / kPageTokens + slot], 0), a.n_pages - 1) : -1;
        if (slot < 8) {
            const int vals[8] = {req, head, t0, t1, f_off[req] + s_off[req] + (is_full ? cj : nfull + cj), t1 == n, 0, 0};
            rec[16 + slot] = vals[slot];
        }
    }
}

__global__ __launch_bounds__(256) void attn_plan_kernel(PlanArgs a) { attn_plan_block(a, blockIdx.x, gridDim.x); }

static PlanArgs plan_args(const AttnPlan& plan, const int32_t* n_or_len, int len_plus, int batch, const int32_t* page_tables,
                          int max_pages, int n_pages, int Hkv, int& blocks) {
    const long long items = (long long)plan.max_chunks * Hkv;
    blocks = (int)max(1LL, min((items + 15) / 16, 1024LL));
    return PlanArgs{n_or_len, page_tables, plan.chunk_off, plan.full_off, plan.records, len_plus, batch,
                    max_pages, n_pages, Hkv};
}

hipError_t launch_attn_plan(const AttnPlan& plan, const int32_t* n_or_len, int len_plus, int batch,
                            const int32_t* page_tables, int max_pages, int n_pages, int Hkv, hipStream_t st) {
    if (batch > 1024) return hipErrorInvalidValue;
    int blocks;
    const PlanArgs a = plan_args(plan, n_or_len, len_plus, batch, page_tables, max_pages, n_pages, Hkv, blocks);
    hipLaunchKernelGGL(attn_plan_kernel, dim3(blocks), dim3(256), 0, st, a);
    return hipGetLastError();
}

// ---------------- first launch of a decode step ----------------
// What depends on the step's inputs alone, in one launch instead of four (each costs 3 to 5 us beside its work):
// workgroups 0 .. batch - 1 gather a row's embedding and its rotary table, the others make the attention plan.
__global__ __launch_bounds__(256) void step_begin_kernel(EmbedRope e, PlanArgs a, LayersZero z) {
    if (blockIdx.x == gridDim.x - 1)
        for (int i = threadIdx.x; i <= z.n; i += 256) {
            if (i < z.n) z.p[i] = 0;
            else if (z.lost) *z.lost = 0;
        }
    if ((int)blockIdx.x < a.batch) embed_rope_row(e, blockIdx.x);
    else attn_plan_block(a, blockIdx.x - a.batch, gridDim.x - a.batch);
}

hipError_t launch_step_begin(const sun_model_cfg& cfg, const void* embed, const int32_t* tokens, const int32_t* seq_lens, int batch,
                             float* x, float* table, const AttnPlan& plan, const int32_t* page_tables, int max_pages,
                             int n_pages, LayersZero zero, hipStream_t st) {
    if (batch > 1024) return hipErrorInvalidValue;
    int blocks;
    const PlanArgs a = plan_args(plan, seq_lens, 1, batch, page_tables, max_pages, n_pages, cfg.n_kv_heads, blocks);
    hipLaunchKernelGGL(step_begin_kernel, dim3(batch + blocks), dim3(256), 0, st, make_embed_rope(cfg, embed, tokens, seq_lens, 0, x, table), a, zero);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// split kernel, matrix-core variant
// ---------------------------------------------------------------------------------
template <int D, int G, KRead K_READ>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_split_kernel(AttnArgs a) {
    __shared__ int list_cursor;
    attn_split_items<D, G, false, K_READ>(a, blockIdx.x, gridDim.x, threadIdx.x & 63, &list_cursor, [] {});
}

// One dim's share of a page: acc + p[0] v[0] + ... in the order of the tokens, the first `count` of them (slots past the end may hold
// anything), vnew in the place of token `fresh`.  All but the last page of a chunk take the sixteen without a question; with
// one asked at every token, and its p read from LDS behind it, 64 tokens took 3 us.
__device__ __forceinline__ float page_dot(float acc, const float* p, const u32x4 (&v)[2], int count, int fresh, float vnew) {
    f32x4 q[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) q[i] = reinterpret_cast<const f32x4*>(p)[i];
    const auto value = [&](int e) {
        const uint32_t w = v[e >> 3][(e & 7) >> 1];
        return e & 1 ? bf16_hi(w) : bf16_lo(w);
    };
    if (count >= kPageTokens && fresh >= kPageTokens) {
#pragma unroll
        for (int e = 0; e < kPageTokens; ++e) acc = fmaf(q[e >> 2][e & 3], value(e), acc);
    } else {
#pragma unroll
        for (int e = 0; e < kPageTokens; ++e) {
            const float more = fmaf(q[e >> 2][e & 3], e == fresh ? vnew : value(e), acc);
            acc = e < count ? more : acc;
        }
    }
    return acc;
}

// ---------------------------------------------------------------------------------
// split kernel, fp32 vector-ALU variant (parity configuration); a workgroup of four waves per item
// ---------------------------------------------------------------------------------
// Bound by latency: an item is at most a few KiB.  A wave per query head in both products (a token's score, then a dim's
// sum over the tokens, one thread and one order of sums each), with all of a thread's loads in flight: a K row, a page's
// 16 tokens of V^T.  With one wave walking its item element by element the launch of the tiny configuration (8 requests
// of 16 to 128 tokens) took 28.9 us; this one takes 7.1.
template <int D>
__global__ __launch_bounds__(256) void attn_split_f32_kernel(AttnArgs a, int G) {
    __shared__ __attribute__((aligned(16))) float qs[8 * D], sc[8][CH];
    __shared__ int pages[CH / kPageTokens];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int total_items = a.chunk_off[a.batch] * a.Hkv;
    for (int item = blockIdx.x; item < total_items; item += gridDim.x) {
        const int32_t* rec = a.records + (size_t)item * kRecInts;
        const int req = rec[16], head = rec[17], t0 = rec[18], t1 = rec[19], chunk_idx = rec[20], cnt = t1 - t0;
        const uint16_t* kb = a.kbase + head * a.k_head;
        const uint16_t* vb = a.vbase + head * a.v_head;
        __syncthreads();  // the previous item's last reads of LDS
        if (tid < CH / kPageTokens) pages[tid] = max(rec[tid], 0);  // the record's page ids are clamped into the pool already
        const float* qp = a.q + ((size_t)req * a.Hq + head * G) * D;
        for (int i = tid; i < G * D; i += 256) qs[i] = qp[i];
        __syncthreads();
        // scores: lane <-> token, wave <-> head
        for (int tt = lane; tt < cnt; tt += 64) {
            const u32x4* kr = reinterpret_cast<const u32x4*>(kb + (int64_t)pages[tt / kPageTokens] * a.k_page + (tt % kPageTokens) * D);
            u32x4 kw[D / 8];
#pragma unroll
            for (int i = 0; i < D / 8; ++i) kw[i] = kr[i];
            for (int g = wave; g < G; g += 4) {
                const f32x4* qg = reinterpret_cast<const f32x4*>(qs + g * D);
                float acc = 0.f;
#pragma unroll
                for (int i = 0; i < D / 8; ++i) {
                    const f32x4 q0 = qg[2 * i], q1 = qg[2 * i + 1];
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        acc = fmaf(w < 2 ? q0[2 * w] : q1[2 * w - 4], bf16_lo(kw[i][w]), acc);
                        acc = fmaf(w < 2 ? q0[2 * w + 1] : q1[2 * w - 3], bf16_hi(kw[i][w]), acc);
                    }
                }
                sc[g][tt] = acc * a.qscale;
            }
        }
        __syncthreads();
        float* pbase = a.partial + ((size_t)chunk_idx * a.Hq + head * G) * (D + 2);
        for (int g = wave; g < G; g += 4) {
            float mx = -INFINITY;
            for (int tt = lane; tt < cnt; tt += 64) mx = fmaxf(mx, sc[g][tt]);
            mx = wave_max(mx);
            float sum = 0.f;
            for (int tt = lane; tt < cnt; tt += 64) {
                const float p = exp2f(sc[g][tt] - mx);
                sc[g][tt] = p;
                sum += p;
            }
            sum = wave_sum(sum);
            if (lane == 0) {
                pbase[(size_t)g * (D + 2) + D] = mx;
                pbase[(size_t)g * (D + 2) + D + 1] = sum;
            }
        }
        __syncthreads();
        // output: lane <-> dim, wave <-> head; 16 tokens of a page are 32 contiguous bytes of V^T
        for (int g = wave; g < G; g += 4)
            for (int j = lane; j < D; j += 64) {
                float acc = 0.f;
                for (int p0 = 0; p0 * kPageTokens < cnt; p0 += 4) {
                    u32x4 v[4][2];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int pg = min(p0 + i, (cnt - 1) / kPageTokens);
                        const u32x4* vr = reinterpret_cast<const u32x4*>(vb + (int64_t)pages[pg] * a.v_page + j * kPageTokens);
                        v[i][0] = vr[0];
                        v[i][1] = vr[1];
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int from = (p0 + i) * kPageTokens;
                        if (from < cnt) acc = page_dot(acc, &sc[g][from], v[i], cnt - from, kPageTokens, 0.f);
                    }
                }
                pbase[(size_t)g * (D + 2) + j] = acc;
            }
    }
}

// ---------------------------------------------------------------------------------
// fp32, short tables: rotation, append, attention over all chunks and their merge in one launch
// ---------------------------------------------------------------------------------
// Bound by latency like the launches it replaces (rope_append_kernel, attn_split_f32_kernel, attn_combine_kernel: three of
// a layer's seven).  A workgroup per request and KV head takes the new position's heads out of the q/k/v product, appends K
// and V, walks the request's chunks (a wave per chunk and query head, partial results in LDS) and merges them.  Every sum has
// the order it has there, so the results are theirs bit for bit.  The compiler's registers count: more workgroups than compute units are two or more
// on one.  With a wave's first keys and values requested in front of the new position's heads, and the new key selected instead of branched
// to (248 registers with 64 dims, 256 and 16 in memory with 128), a step of the tiny shape with 8 / 128 / 256 requests of up to 128 / 370 / 370 tokens took 57 / 112 / 159
// us, without (75 and 87 registers) 57 / 110 / 144; 4 query heads of 128 dims, 200 requests of 60 tokens 293 -> 280.
// A request is a few workgroups', so longer tables stay with the launches that spread it.  How long depends on a workgroup's share, chunks x
// query heads x dims at 64 positions a chunk.  Two KV heads, hidden 512, 8 requests, tables of 64 / 128 / 192 / 256 / 384 positions full, three launches -> this (us a
// step): 2 query heads of 128 each 79 / 85 / 86 / 86 / 88 -> 70 / 80 / 83 / 84 / 94, 4 of 64 79 / 78 / 77 / 77 / 82 -> 67 / 69 / 73 / 75 / 87, 8 of 64 92 / 89 / 95 /
// 99 / 97 -> 81 / 85 / 97 / 107 / 118, 4 of 128 94 / 97 / 99 / 101 / 101 -> 86 / 93 / 101 / 109 / 121, 8 of 128 120 / 121 / 121 / 121 / 122 -> 110 / 122 / 134 /
// 146 / 171 (1 and 32 requests the same way); hence kShortShare.  From 128 requests on up to twice that share is faster here too (4 of 128, 256 requests,
// 256 positions 376 -> 356), 8 of 128 is even.
// Not for a prefill block, where a row attends to entries that other rows of the launch append.
constexpr int kShortPart = (kShortTokens / kAttnSmall) * 8 * 130;   // floats of LDS for partial results: chunks, query heads, dims + 2

struct ShortArgs {
    const float *qkv, *table, *bq, *bk, *bv, *qn, *kn;   // biases and head-norm gains may be NULL
    const int32_t *seq_lens, *page_tables;
    uint16_t *kbase, *vbase;                             // of the layer
    int64_t k_page, k_head, v_page, v_head;
    float* out;                                          // [batch, Hq * D]
    int batch, Hq, Hkv, max_pages, n_pages;
    float eps, qscale;
};

template <int D>
__global__ __launch_bounds__(512) void attn_short_f32_kernel(ShortArgs a) {
    constexpr int W = 8, half = D / 2;
    __shared__ __attribute__((aligned(16))) float qs[8 * D], sc[W][CH], part[kShortPart];
    __shared__ __attribute__((aligned(16))) uint16_t kv[2][D];   // the new entry
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, kh = blockIdx.x, b = blockIdx.y, G = a.Hq / a.Hkv;
    // lengths and page ids are validated on the host under SUN_VALIDATE; clamp so bad input cannot fault
    const int L = min(max(a.seq_lens[b], 0), a.max_pages * kPageTokens - 1), n = L + 1;
    const int32_t* pt = a.page_tables + (size_t)b * a.max_pages;
    const auto page_of = [&](int p) { return min(max(pt[p], 0), a.n_pages - 1); };
    uint16_t *kb = a.kbase + (int64_t)kh * a.k_head, *vb = a.vbase + (int64_t)kh * a.v_head;
    for (int t = wave; t < G + 2; t += W) {                 // a wave per head; lane j holds elements j and j + D / 2
        const int hh = t < G ? kh * G + t : t == G ? a.Hq + kh : a.Hq + a.Hkv + kh, j = lane;
        const bool act = j < half;
        const float* src = a.qkv + ((size_t)b * (a.Hq + 2 * a.Hkv) + hh) * D;
        float lo = 0.f, hi = 0.f;
        if (act) {
            lo += src[j];
            hi += src[j + half];
        }
        if (a.bq && act) {
            const float* bias = t < G ? a.bq : t == G ? a.bk : a.bv;
            const int h0 = (t < G ? hh : kh) * D;
            lo += bias[h0 + j];
            hi += bias[h0 + j + half];
        }
        if (a.qn && t <= G) {
            const float ss = wave_sum(lo * lo + hi * hi);
            const float r = 1.0f / sqrtf(ss / (float)D + a.eps);
            if (act) {
                const float* g = t < G ? a.qn : a.kn;
                lo = lo * r * g[j];
                hi = hi * r * g[j + half];
            }
        }
        if (!act) continue;
        if (t <= G) {
            const float c = a.table[((size_t)b * half + j) * 2], sn = a.table[((size_t)b * half + j) * 2 + 1];
            const float rl = lo * c - hi * sn, rh = hi * c + lo * sn;
            lo = rl;
            hi = rh;
        }
        if (t < G) {
            qs[t * D + j] = lo;
            qs[t * D + j + half] = hi;
        } else {
            const uint16_t l16 = f32_to_bf16_bits(lo), h16 = f32_to_bf16_bits(hi);
            const int64_t page = page_of(L / kPageTokens), slot = L % kPageTokens;
            kv[t - G][j] = l16;
            kv[t - G][j + half] = h16;
            if (t == G) {
                kb[page * a.k_page + slot * D + j] = l16;
                kb[page * a.k_page + slot * D + j + half] = h16;
            } else {
                vb[page * a.v_page + (int64_t)j * kPageTokens + slot] = l16;
                vb[page * a.v_page + (int64_t)(j + half) * kPageTokens + slot] = h16;
            }
        }
    }
    int n_full, n_small, ch;
    attn_chunking(n, a.batch, a.Hkv, n_full, n_small, ch);
    const int nc = n_full + n_small;
    __syncthreads();
    for (int task = wave; task < nc * G; task += W) {       // a wave per chunk and query head
        const int ci = task / G, g = task % G;
        const int t0 = ci < n_full ? ci * ch : n_full * ch + (ci - n_full) * kAttnSmall, t1 = ci < n_full ? t0 + ch : min(n, t0 + kAttnSmall);
        const int cnt = t1 - t0;
        float* s = sc[wave];
        float mx = -INFINITY;
        for (int tt = lane; tt < cnt; tt += 64) {           // scores: lane <-> token; the new one's K comes from LDS
            const int pos = t0 + tt;
            u32x4 kw[D / 8];
            if (pos == L) {
                asm volatile("");                           // a branch: as selects the entry takes registers beside every key's
#pragma unroll
                for (int i = 0; i < D / 8; ++i) kw[i] = reinterpret_cast<const u32x4*>(kv[0])[i];
            } else {
                const u32x4* kr = reinterpret_cast<const u32x4*>(kb + (int64_t)page_of(pos / kPageTokens) * a.k_page + (pos % kPageTokens) * D);
#pragma unroll
                for (int i = 0; i < D / 8; ++i) kw[i] = kr[i];
            }
            const f32x4* qg = reinterpret_cast<const f32x4*>(qs + g * D);
            float acc = 0.f;
#pragma unroll
            for (int i = 0; i < D / 8; ++i) {
                const f32x4 q0 = qg[2 * i], q1 = qg[2 * i + 1];
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    acc = fmaf(w < 2 ? q0[2 * w] : q1[2 * w - 4], bf16_lo(kw[i][w]), acc);
                    acc = fmaf(w < 2 ? q0[2 * w + 1] : q1[2 * w - 3], bf16_hi(kw[i][w]), acc);
                }
            }
            const float v = acc * a.qscale;
            s[tt] = v;
            mx = fmaxf(mx, v);
        }
        mx = wave_max(mx);
        float sum = 0.f;
        for (int tt = lane; tt < cnt; tt += 64) {
            const float p = exp2f(s[tt] - mx);
            s[tt] = p;
            sum += p;
        }
        sum = wave_sum(sum);
        float* pb = part + task * (D + 2);
        if (lane == 0) {
            pb[D] = mx;
            pb[D + 1] = sum;
        }
        __builtin_amdgcn_wave_barrier();                    // the lanes' scores are read by all of them; a wave's LDS accesses are in order
        for (int j = lane; j < D; j += 64) {                // output: lane <-> dim
            const float vnew = bf16_bits_to_f32(kv[1][j]);
            float acc = 0.f;
            for (int p0 = 0; p0 * kPageTokens < cnt; p0 += 4) {
                u32x4 v[4][2];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int pg = min(p0 + i, (cnt - 1) / kPageTokens);
                    const u32x4* vr = reinterpret_cast<const u32x4*>(vb + (int64_t)page_of(t0 / kPageTokens + pg) * a.v_page + j * kPageTokens);
                    v[i][0] = vr[0];
                    v[i][1] = vr[1];
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int from = (p0 + i) * kPageTokens;
                    if (from < cnt) acc = page_dot(acc, s + from, v[i], cnt - from, L - t0 - from, vnew);
                }
            }
            pb[j] = acc;
        }
    }
    __syncthreads();
    for (int i = tid; i < G * D; i += 512) {                // merged in chunk order, the maximum moves once per eight chunks
        const int g = i / D, j = i % D;
        float M = -INFINITY, num = 0.f, den = 0.f;
        for (int c8 = 0; c8 < nc; c8 += 8) {
            const int c9 = min(nc, c8 + 8);
            float top = M;
            for (int c = c8; c < c9; ++c) top = fmaxf(top, part[(c * G + g) * (D + 2) + D]);
            const float s8 = exp2f(M - top);
            num *= s8;
            den *= s8;
            M = top;
            for (int c = c8; c < c9; ++c) {
                const float* pb = part + (c * G + g) * (D + 2);
                const float wk = exp2f(pb[D] - M);
                den = fmaf(wk, pb[D + 1], den);
                num = fmaf(wk, pb[j], num);
            }
        }
        a.out[((size_t)b * a.Hq + kh * G + g) * D + j] = num / den;
    }
}

bool attn_short_f32(const sun_model_cfg& c, int max_pages) {
    // every chunk but a request's last covers at least kAttnSmall positions
    const long long positions = (long long)max_pages * kPageTokens, chunks = (positions + kAttnSmall - 1) / kAttnSmall;
    return c.n_q_heads / c.n_kv_heads <= 8 && c.head_dim <= 128 && positions <= kShortTokens &&
           chunks * (c.n_q_heads / c.n_kv_heads) * c.head_dim <= kShortShare;
}

hipError_t launch_attn_short_f32(const KvPool& pool, int layer, const float* qkv, const float* table, const int32_t* seq_lens, const int32_t* page_tables,
                                 int max_pages, int batch, const LayerW& w, float* out, hipStream_t st) {
    const sun_model_cfg& c = pool.cfg;
    const sun_kv_layout& L = pool.lay;
    if (!attn_short_f32(c, max_pages) || L.k_dim != 1 || L.k_token != c.head_dim || L.v_token != 1 || L.v_dim != kPageTokens) return hipErrorInvalidValue;
    const auto f = [](bool on, const void* p) { return on ? (const float*)p : nullptr; };
    const ShortArgs a{qkv, table, f(c.qkv_bias, w.bq), f(c.qkv_bias, w.bk), f(c.qkv_bias, w.bv), f(c.qk_norm, w.qn), f(c.qk_norm, w.kn), seq_lens, page_tables,
                      pool.base + L.k_off + (int64_t)layer * L.k_layer, pool.base + L.v_off + (int64_t)layer * L.v_layer, L.k_page, L.k_head, L.v_page, L.v_head,
                      out, batch, c.n_q_heads, c.n_kv_heads, max_pages, (int)L.n_pages, c.rms_eps, kLog2e / sqrtf((float)c.head_dim)};
    const dim3 grid(c.n_kv_heads, batch);
    if (c.head_dim == 64) hipLaunchKernelGGL(attn_short_f32_kernel<64>, grid, dim3(512), 0, st, a);
    else if (c.head_dim == 128) hipLaunchKernelGGL(attn_short_f32_kernel<128>, grid, dim3(512), 0, st, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// What fits the memory-side cache (256 MB) from one step to the next is read through it: K of all layers, beside the weights where
// those stay there too (bf16, no more than kStreamWeightBytes).  Streamed -> through the caches, us a step: hidden 512, 2 layers, 20 MB of weights, K of
// 107 / 184 MB 209 -> 202 / 239 -> 230; hidden 1024, 4 layers, 120 MB, K of 41 / 73 / 115 / 131 MB 216 -> 211 / 415 -> 406 / 232 -> 234 / 272 -> 276; hidden
// 1024, 8 layers, 197 MB, K of 20 / 37 MB 405 -> 402 / 749 -> 757; weights past the caches: hidden 2048, 4 layers, K of 131 / 307 MB 380 -> 367 / 737 -> 737,
// hidden 4096, 2 layers, 184 / 524 MB 394 -> 385 / 807 -> 805, 32 query heads on 4, hidden 2048, 246 / 393 MB 452 -> 449 / 518 -> 527.  With 4-bit weights, which are
// never streamed, K of 7 to 246 MB 272 -> 278 up to 399 -> 409.  In the one launch of all layers K is always streamed: never slower than
// the cached loads of the operand as it lies that stood there before, and by turns 1 % behind and 8 % ahead of cached rows.
// In rows or in place: turning the rows costs the vector ALU, in place an instruction takes 16 bytes of each of 64 half lines.  Steps take rows, in place is
// 1 to 2 % slower there up to some 60 MB of K (and as much faster at 184); attention alone, 256 requests of 400 / 700 tokens, 8 query heads on 2, two layers 65.8 -> 60.9 / 86 ->
// 81 us, 64 of 1000, 32 on 8, one layer 55.5 -> 52.9.
KRead attn_k_read(const sun_model_cfg& c, const Weights* W, long long tokens) {
    constexpr size_t kKept = (size_t)224 << 20;
    const size_t beside = !W || W->layers[0].qkv.stream ? 0 : W->packed;
    if ((W && W->quant) || beside + (size_t)tokens * c.n_kv_heads * c.head_dim * 2 * c.n_layers > kKept) return K_STREAMED;
    return W ? K_ROWS : K_IN_PLACE;
}

template <int D, KRead K_READ>
static hipError_t launch_split_d(const AttnArgs& a, int G, int grid, hipStream_t st) {
    switch (G) {
#define SUN_CASE(g) \
    case g: hipLaunchKernelGGL((attn_split_kernel<D, g, K_READ>), dim3(grid), dim3(512), 0, st, a); break;
        SUN_CASE(1) SUN_CASE(2) SUN_CASE(3) SUN_CASE(4) SUN_CASE(5) SUN_CASE(6) SUN_CASE(7) SUN_CASE(8)
#undef SUN_CASE
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_attn_split(const KvPool& pool, int layer, const AttnPlan& plan, const float* q,
                             const int32_t* page_tables, int max_pages, const int32_t* n_or_len, int len_plus,
                             int batch, int total_chunks_hint, int full_chunks_hint, KRead k_read, bool f32_exact, hipStream_t st) {
    const sun_model_cfg& c = pool.cfg;
    const sun_kv_layout& L = pool.lay;
    const int D = c.head_dim, G = c.n_q_heads / c.n_kv_heads;
    if (L.k_dim != 1 || L.k_token != D || L.v_token != 1 || L.v_dim != kPageTokens) return hipErrorInvalidValue;
    AttnArgs a = make_attn_args(pool, layer, plan, q, page_tables, max_pages, n_or_len, len_plus, batch);
    const long long chunks = total_chunks_hint >= 0 ? total_chunks_hint : plan.max_chunks;
    const long long items = chunks * c.n_kv_heads;
    if (f32_exact) {
        if (G > 8) return hipErrorInvalidValue;
        const int grid = (int)max(1LL, min(items, 4096LL));
        if (D == 64) hipLaunchKernelGGL(attn_split_f32_kernel<64>, dim3(grid), dim3(256), 0, st, a, G);
        else if (D == 128) hipLaunchKernelGGL(attn_split_f32_kernel<128>, dim3(grid), dim3(256), 0, st, a, G);
        else return hipErrorInvalidValue;
        return hipGetLastError();
    }
    // persistent workgroups of 8 waves, one per compute unit (fewer only when there are fewer
    // items than waves)
    // the item counts travel as kernel arguments when the host knows them: one dependent load less before a
    // wave's first request for K and V
    if (full_chunks_hint >= 0 && total_chunks_hint >= 0) {
        a.n_full_items = full_chunks_hint * c.n_kv_heads;
        a.total_items = total_chunks_hint * c.n_kv_heads;
    }
    const int grid = (int)max(1LL, min((items + 7) / 8, 256LL));
    if (D == 64) return launch_split_d<64, K_IN_PLACE>(a, G, grid, st);
    if (D != 128) return hipErrorInvalidValue;
    switch (k_read) {
    case K_STREAMED: return launch_split_d<128, K_STREAMED>(a, G, grid, st);
    case K_ROWS: return launch_split_d<128, K_ROWS>(a, G, grid, st);
    case K_IN_PLACE: return launch_split_d<128, K_IN_PLACE>(a, G, grid, st);
    }
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------------
// combine: merge the chunk partials of a request in chunk order
// ---------------------------------------------------------------------------------
struct CombineArgs {
    const int32_t* chunk_off;  // NULL: every request has `uniform` chunks
    const float* partial;
    float* out_f32;
    uint16_t* out_tiled;
    float* qscale;
    int Hq, D, batch, out_mb, uniform;
};

// A workgroup merges 128 columns of a request: one head of 128 dims or two of 64, each wave for itself.  Chunks are added in
// token order under a running maximum that moves once per eight chunks.  Bound by the latency of the partials, which the
// split kernel has just written.  Up to eight chunks every thread reads all of them at once.  Beyond that 64 chunks' maxima and
// sums are read at once, a lane per chunk, and their weights and the eights' rescaling factors computed there, so that the
// outputs' loads depend on nothing but each other's order and sixteen of them are in flight per thread.  With eight
// chunks a round throughout, each round's loads behind the rescaling of the one before: 8B shape, 16 / 256 requests 6.4 -> 5.3 /
// 21.7 -> 17.0 us, 14B shape, 24 requests of 17 k tokens 24.4 -> 17.0; a lane per chunk throughout: 1000 requests of up to
// 400 tokens 48 instead of 37.
__global__ __launch_bounds__(128) void attn_combine_kernel(CombineArgs a) {
    const int b = blockIdx.y, col = blockIdx.x * 128 + threadIdx.x, lane = threadIdx.x & 63;
    const int h = col / a.D, j = col % a.D;   // a wave's 64 columns are of one head
    const int c0 = a.chunk_off ? a.chunk_off[b] : b * a.uniform, c1 = a.chunk_off ? a.chunk_off[b + 1] : c0 + a.uniform;
    const int n = c1 - c0;
    const size_t stride = (size_t)a.Hq * (a.D + 2);
    const float* p = a.partial + (size_t)c0 * stride + (size_t)h * (a.D + 2);
    float M = -INFINITY, num = 0.f, den = 0.f;
    if (n <= 8) {                             // one group: every thread reads all of it
        float m8[8], l8[8], o8[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float* pc = p + min(i, n - 1) * stride;
            m8[i] = pc[a.D];
            l8[i] = pc[a.D + 1];
            o8[i] = pc[j];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) M = fmaxf(M, m8[i]);
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (i < n) {
                const float w = exp2f(m8[i] - M);
                den = fmaf(w, l8[i], den);
                num = fmaf(w, o8[i], num);
            }
    } else {
        for (int cb = 0; cb < n; cb += 64) {
            const int c = cb + lane, cnt = min(n - cb, 64);
            const float m = c < n ? p[c * stride + a.D] : -INFINITY, l = c < n ? p[c * stride + a.D + 1] : 0.f;
            float prev;                           // maximum up to the start and to the end of the lane's eight
            const float top = wave_octet_max(m, M, prev);
            const float w = c < n ? exp2f(m - top) : 0.f, sc = exp2f(prev - top);
            M = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(top), 63));
            const float* pj = p + (size_t)cb * stride + j;
            for (int k0 = 0; k0 < cnt; k0 += 16) {
                float o[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) o[i] = pj[min(k0 + i, cnt - 1) * stride];
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (k0 + i < cnt) {
                        if (i % 8 == 0) {
                            const float s = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(sc), k0 + i));
                            num *= s;
                            den *= s;
                        }
                        const float wk = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w), k0 + i));
                        den = fmaf(wk, __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(l), k0 + i)), den);
                        num = fmaf(wk, o[i], num);
                    }
            }
        }
    }
    const float v = num / den;
    if (a.out_f32) a.out_f32[(size_t)b * a.Hq * a.D + col] = v;
    if (a.out_tiled && !a.qscale) {
        uint16_t lo;
        const uint16_t hi = split_bf16(v, lo);
        a.out_tiled[atile_elem(ATile{a.out_mb}, 0, b, col)] = hi;
        a.out_tiled[atile_elem(ATile{a.out_mb}, 1, b, col)] = lo;
    }
    if (a.out_tiled && a.qscale) {
        // fixed-point tile of the 4-bit O projection: the workgroup's 128 columns are one group
        __shared__ float red_max[2];
        __shared__ int red_sum[2];
        const float wm = wave_max(fabsf(v));
        if ((threadIdx.x & 63) == 0) red_max[threadIdx.x >> 6] = wm;
        __syncthreads();
        const float am = fmaxf(red_max[0], red_max[1]);
        const int xi = (int)rintf(v * qtile_inv(am));
        const int l = ((xi + 128) & 255) - 128, hq = (xi - l) >> 8;
        uint8_t* tile = reinterpret_cast<uint8_t*>(a.out_tiled);
        tile[qtile_unit(ATile{a.out_mb}, 0, b, col >> 4) * 16 + (col & 15)] = (uint8_t)(hq & 255);
        tile[qtile_unit(ATile{a.out_mb}, 1, b, col >> 4) * 16 + (col & 15)] = (uint8_t)(l & 255);
        int sum = xi;
        sum = wave_sum(sum);
        if ((threadIdx.x & 63) == 0) red_sum[threadIdx.x >> 6] = sum;
        __syncthreads();
        if (threadIdx.x == 0)
            reinterpret_cast<float2*>(a.qscale)[(size_t)blockIdx.x * (a.out_mb * 32) + b] =
                float2{am / kQMax, __int_as_float(red_sum[0] + red_sum[1])};
    }
}

static hipError_t launch_combine(const sun_model_cfg& cfg, const int32_t* chunk_off, int uniform, const float* partial,
                                 int batch, float* out_f32, void* out_tiled, float* qscale, hipStream_t st) {
    CombineArgs a{};
    a.chunk_off = chunk_off;
    a.uniform = uniform;
    a.partial = partial;
    a.out_f32 = out_f32;
    a.out_tiled = (uint16_t*)out_tiled;
    a.qscale = qscale;
    a.Hq = cfg.n_q_heads;
    a.D = cfg.head_dim;
    a.batch = batch;
    a.out_mb = atile_for_rows(batch).MB;
    const int cols = cfg.n_q_heads * cfg.head_dim;
    if (cols % 128) return hipErrorInvalidValue;
    hipLaunchKernelGGL(attn_combine_kernel, dim3(cols / 128, batch), dim3(128), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_attn_combine(const sun_model_cfg& cfg, const AttnPlan& plan, int batch, float* out_f32,
                               void* out_tiled, float* qscale, hipStream_t st) {
    return launch_combine(cfg, plan.chunk_off, 0, plan.partial, batch, out_f32, out_tiled, qscale, st);
}

// ---------------------------------------------------------------------------------
// prefill: the causal attention of a block of consecutive positions of one request
// ---------------------------------------------------------------------------------
// Eq. 2's attention for `rows` rows at once.  A wave owns 32 query rows of one head, a workgroup four waves (the heads of a
// group, or heads of neighbouring row blocks, all of one KV head), and the K and V of 32 keys pass through LDS once for
// all of them: the row-by-row kernel above reads the whole cache once per row (1024 rows of the 8B shape: 240 us a layer
// and 38 for its combine, here 53; 3000 rows behind 1003 keys: 2670 us a layer and 180, here 366).  Bound by the
// matrix cores and the softmax between them (32 instructions of 32 cycles and some 200 vector instructions per wave
// and tile, two waves per SIMD); both planes of q and of P, as in a decode step.
//   S^T[key, row] = K . q^T, so that a lane holds 16 scores of one row and its running maximum needs one exchange;
//   O^T[dim, row] += V^T . P^T, whose second operand is exactly the scores the lane holds, and whose rescaling needs no
//   exchange at all.  K and V go from memory straight into three LDS slots, two tiles ahead.
// blockIdx.x is the KV head: with eight of them each XCD keeps one head's K and V in its own L2.
struct PrefillAttnArgs {
    const uint16_t* kbase;
    const uint16_t* vbase;
    int64_t k_page, k_head, v_page, v_head;
    const float* q;              // [rows, Hq*D], rotated
    const int32_t* page_table;   // the request's row
    uint16_t* out;               // two-plane tile of the O projection [rows, Hq*D] (one split), or
    float* partial;              // [rows][splits][Hq][D + 2] (o[D], m, l)
    int rows, first, Hq, G, n_pages, mb, tiles_per_split;
    float qscale;                // log2(e) / sqrt(D)
};

template <int D>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_prefill_kernel(PrefillAttnArgs a) {
    constexpr int NWV = 4;
    constexpr int KS = D / 16;              // k-steps of the score product
    constexpr int DB = D / 32;              // 32-row blocks of the output (dims)
    constexpr int OCT = D / 8;              // 16-byte units of a K row
    constexpr int KI = 32 * OCT / 64;       // fetch instructions (1 KiB) of a tile's K; as many for its V
    constexpr int PER = (2 * KI + NWV - 1) / NWV;
    constexpr int TILE_UNITS = 2 * KI * 64; // K, then V: 16 KiB at D = 128
    constexpr int NBUF = 3;
    __shared__ u32x4 lds[NBUF * TILE_UNITS];

    const int tid = threadIdx.x, lane = tid & 63, c32 = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // A wave's item is (32 rows, query head of the group); four consecutive items share a workgroup.  The longest start first.
    const int n_items = (a.rows + 31) / 32 * a.G, item0 = (int)(gridDim.y - 1 - blockIdx.y) * NWV, item = item0 + wave;
    const int blk = item / a.G, hkv = blockIdx.x, hq = hkv * a.G + item % a.G;
    const int row = blk * 32 + c32;                                // this lane's query row
    const int qpos = a.first + row;
    const int total = a.first + a.rows;                            // positions that hold a key
    const int my_first = a.first + blk * 32;                       // first position of the wave's rows
    const auto tiles_of = [&](int bl) { return (a.first + min(a.rows, bl * 32 + 32) - 1) / 32 + 1; };
    const int t_begin = blockIdx.z * a.tiles_per_split;            // this split's tiles of 32 keys
    const int t_end = min(tiles_of(min(item0 + NWV - 1, n_items - 1) / a.G), t_begin + a.tiles_per_split);
    const int my_end = item < n_items ? min(tiles_of(blk), t_end) : 0;

    // q as the second operand (columns = query rows): 8 dims per lane and k-step, hi and lo bf16
    bf16x8 qhi[KS], qlo[KS];
    {
        const float* qp = a.q + ((size_t)min(row, a.rows - 1) * a.Hq + hq) * D + h * 8;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const f32x4 v0 = *reinterpret_cast<const f32x4*>(qp + s * 16), v1 = *reinterpret_cast<const f32x4*>(qp + s * 16 + 4);
            const float x[8] = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
            u32x4 hi, lo;
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                uint32_t ph, pl;
                split_pair(x[2 * p] * a.qscale, x[2 * p + 1] * a.qscale, ph, pl);
                hi[p] = ph;
                lo[p] = pl;
            }
            qhi[s] = __builtin_bit_cast(bf16x8, hi);
            qlo[s] = __builtin_bit_cast(bf16x8, lo);
        }
    }
    // Fetch instruction j of a tile.  K (j < KI): LDS row rho holds the token whose score the MFMA puts into row rho; rho
    // = 8 i + 4 h + e belongs to lane half h, which is to hold eight consecutive tokens of each page for the second
    // product: token 8 h + 4 i + e (i = 0, 1), the same 16 further on for the second page.  The 16-byte units of a row are
    // exchanged by the row's number, so that a fragment read meets every bank once.  V: fragment order, (page, 32-dim block)
    // per instruction.
    const uint16_t *kb = a.kbase + hkv * a.k_head, *vb = a.vbase + hkv * a.v_head;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) u32x4*)lds;
    int pg_sel[PER];
    uint32_t lane_off[PER];
    bool is_k[PER];
    uint32_t dst[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int j = min(wave + i * NWV, 2 * KI - 1);             // past the last one: that one again, the same bytes
        is_k[i] = j < KI;
        if (is_k[i]) {
            const int rho = j * (64 / OCT) + lane / OCT, u = lane % OCT;
            const int r16 = rho & 15, tok = 8 * ((r16 >> 2) & 1) + 4 * (r16 >> 3) + (r16 & 3);
            pg_sel[i] = (j * (64 / OCT)) >> 4;
            lane_off[i] = (tok * OCT + (u ^ (rho & (OCT - 1)))) * 16;
        } else {
            const int f = j - KI;
            pg_sel[i] = f / DB;
            lane_off[i] = (((f % DB) * 32 + c32) * 2 + h) * 16;
        }
        dst[i] = lds0 + j * 1024;
    }
    uint32_t fill = 0;
    int fill_tile = t_begin;
    auto page_of = [&](int p) {   // past the last page: the last one (its keys are masked)
        return min(max(load_uniform(a.page_table + min(p, (total - 1) / kPageTokens)), 0), a.n_pages - 1);
    };
    int pgA = page_of(2 * t_begin), pgB = page_of(2 * t_begin + 1);
    auto issue = [&]() {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int64_t pg = pg_sel[i] ? pgB : pgA;
            lds_dma16(is_k[i] ? kb + pg * a.k_page : vb + pg * a.v_page, lane_off[i], dst[i] + fill);
        }
        fill = fill + TILE_UNITS * 16 == NBUF * TILE_UNITS * 16 ? 0 : fill + TILE_UNITS * 16;
        fill_tile = min(fill_tile + 1, t_end - 1);                 // past the end the last tile again (it is not read)
        pgA = page_of(2 * fill_tile);
        pgB = page_of(2 * fill_tile + 1);
    };

    f32x16 O[DB];
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) O[d][r] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    bool poisoned = false;   // a key this row attends to has a V that is not finite

    if (t_begin < t_end) {
#pragma unroll
        for (int b = 0; b < NBUF - 1; ++b) issue();
    }
    int at = 0;
    for (int t = t_begin; t < t_end; ++t) {
        // tile t has landed for every wave, and every wave is done with tile t - 1: its slot takes tile t + 2
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0xc07f);
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(PER * (NBUF - 2)) : "memory");
        issue();
        if (t < my_end) {
            const u32x4* kt = lds + at * TILE_UNITS;
            const u32x4* vt = kt + KI * 64 + lane;
            f32x16 S;
#pragma unroll
            for (int r = 0; r < 16; ++r) S[r] = 0.f;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const bf16x8 kf = __builtin_bit_cast(bf16x8, kt[c32 * OCT + ((s * 2 + h) ^ (c32 & (OCT - 1)))]);
                S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qhi[s], S, 0, 0, 0);
                S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qlo[s], S, 0, 0, 0);
            }
            // this lane: its query row, keys t*32 + 16 (r >> 3) + 8 h + (r & 7)
            const bool diag = t * 32 + 31 > my_first;
            if (diag) {
#pragma unroll
                for (int r = 0; r < 16; ++r) S[r] = t * 32 + 16 * (r >> 3) + 8 * h + (r & 7) <= qpos ? S[r] : -INFINITY;
            }
            float mloc = S[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) mloc = fmaxf(mloc, S[r]);
            mloc = fmaxf(mloc, lane_xor<32>(mloc));
            // a split may begin behind a row's last key: all its scores are masked then, and its weights have to be zeros
            const float m_new = fmaxf(m_run, mloc), m_use = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);
            m_run = m_new;
            float psum = 0.f;
            bf16x8 phi[2], plo[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                u32x4 hi, lo;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float p0 = __builtin_amdgcn_exp2f(S[k * 8 + 2 * e] - m_use), p1 = __builtin_amdgcn_exp2f(S[k * 8 + 2 * e + 1] - m_use);
                    psum += p0 + p1;
                    uint32_t wh, wl;
                    split_pair(p0, p1, wh, wl);
                    hi[e] = wh;
                    lo[e] = wl;
                }
                phi[k] = __builtin_bit_cast(bf16x8, hi);
                plo[k] = __builtin_bit_cast(bf16x8, lo);
            }
            l_run = l_run * alpha + psum;
            if (__any(alpha != 1.f)) {
#pragma unroll
                for (int d = 0; d < DB; ++d)
#pragma unroll
                    for (int r = 0; r < 16; ++r) O[d][r] *= alpha;
            }
            // V of a key that a row does not see meets a zero weight, which only a finite V survives.  In the tiles where
            // that can happen, keys whose V is not finite are left out of the product and mark the rows that do see them;
            // slots past the prompt, which may hold anything, are left out as well.
            uint32_t keep[2][4];
            if (diag) {
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    uint32_t bad = 0;   // this lane half's eight keys of page k
#pragma unroll 1
                    for (int d = 0; d < DB; ++d) {
                        const u32x4 v = vt[(k * DB + d) * 64];
#pragma unroll
                        for (int w = 0; w < 4; ++w) {
                            bad |= (v[w] & 0x00007f80u) == 0x00007f80u ? 1u << (2 * w) : 0u;
                            bad |= (v[w] & 0x7f800000u) == 0x7f800000u ? 2u << (2 * w) : 0u;
                        }
                    }
#pragma unroll
                    for (int o = 1; o < 32; o <<= 1) bad |= __shfl_xor(bad, o);
                    const int key0 = t * 32 + k * 16;
                    const int held = min(max(total - key0 - 8 * h, 0), 8);   // of the eight, how many hold a key
                    bad |= 0xffu & ~((1u << held) - 1u);
#pragma unroll
                    for (int w = 0; w < 4; ++w)
                        keep[k][w] = (bad >> (2 * w) & 1 ? 0u : 0x0000ffffu) | (bad >> (2 * w + 1) & 1 ? 0u : 0xffff0000u);
                    const uint32_t other = __shfl_xor(bad, 32), both = h ? (bad << 8) | other : bad | (other << 8);
                    poisoned = poisoned || (both & ((1u << min(max(qpos - key0 + 1, 0), 16)) - 1u)) != 0;
                }
            }
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int d = 0; d < DB; ++d) {
                    u32x4 v = vt[(k * DB + d) * 64];
                    if (diag) {
#pragma unroll
                        for (int w = 0; w < 4; ++w) v[w] &= keep[k][w];
                    }
                    const bf16x8 vf = __builtin_bit_cast(bf16x8, v);
                    O[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, phi[k], O[d], 0, 0, 0);
                    O[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, plo[k], O[d], 0, 0, 0);
                }
        }
        at = at + 1 == NBUF ? 0 : at + 1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // nothing is in flight into LDS when the workgroup ends
    const float l_sum = l_run + lane_xor<32>(l_run), l_tot = poisoned ? __builtin_nanf("") : l_sum;
    if (row >= a.rows) return;
    if (a.partial) {
        float* o = a.partial + (((size_t)row * gridDim.z + blockIdx.z) * a.Hq + hq) * (D + 2);
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
            for (int i = 0; i < 8; ++i)   // an even number of floats apart, so 8-byte aligned
                *reinterpret_cast<float2*>(o + d * 32 + (i >> 1) * 8 + h * 4 + (i & 1) * 2) = float2{O[d][i * 2], O[d][i * 2 + 1]};
        if (h == 0) *reinterpret_cast<float2*>(o + D) = float2{m_run, l_tot};
        return;
    }
    const float inv = 1.f / l_tot;
    // lane: row c32, dims 32 d + 8 i + 4 h + 0..3: half of a 16-byte unit per plane
    uint2* out = reinterpret_cast<uint2*>(a.out);
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float y[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = O[d][i * 4 + e] * inv;
            uint2 hi, lo;
            hi.x = pack_bf16(y[0], y[1]);
            hi.y = pack_bf16(y[2], y[3]);
            lo.x = pack_bf16(y[0] - bf16_lo(hi.x), y[1] - bf16_hi(hi.x));
            lo.y = pack_bf16(y[2] - bf16_lo(hi.y), y[3] - bf16_hi(hi.y));
            const int k8 = (hq * D + d * 32) / 8 + i;
            out[atile_unit(ATile{a.mb}, 0, row, k8) * 2 + h] = hi;
            out[atile_unit(ATile{a.mb}, 1, row, k8) * 2 + h] = lo;
        }
}

// Key splits of a prefill block: enough workgroups for the 256 compute units, none of them shorter than eight tiles.
int attn_prefill_splits(const sun_model_cfg& c, int rows, int first) {
    const int G = c.n_q_heads / c.n_kv_heads;
    const int wgs = ((rows + 31) / 32 * G + 3) / 4 * c.n_kv_heads, tiles = (first + rows - 1) / 32 + 1;
    return max(1, min(256 / wgs, tiles / 8));
}

hipError_t launch_attn_prefill(const KvPool& pool, int layer, const float* q, const int32_t* page_table, int first, int rows,
                               int splits, float* partial, void* out_tiled, hipStream_t st) {
    const sun_model_cfg& c = pool.cfg;
    const sun_kv_layout& L = pool.lay;
    const int D = c.head_dim, G = c.n_q_heads / c.n_kv_heads;
    if (L.k_dim != 1 || L.k_token != D || L.v_token != 1 || L.v_dim != kPageTokens || rows < 1 || splits < 1) return hipErrorInvalidValue;
    PrefillAttnArgs a{};
    a.kbase = pool.base + L.k_off + (int64_t)layer * L.k_layer;
    a.vbase = pool.base + L.v_off + (int64_t)layer * L.v_layer;
    a.k_page = L.k_page;
    a.k_head = L.k_head;
    a.v_page = L.v_page;
    a.v_head = L.v_head;
    a.q = q;
    a.page_table = page_table;
    a.out = (uint16_t*)out_tiled;
    a.partial = splits > 1 ? partial : nullptr;
    a.rows = rows;
    a.first = first;
    a.Hq = c.n_q_heads;
    a.G = G;
    a.n_pages = (int)L.n_pages;
    a.mb = atile_for_rows(rows).MB;
    a.tiles_per_split = ((first + rows - 1) / 32 + 1 + splits - 1) / splits;
    a.qscale = kLog2e / sqrtf((float)D);
    const dim3 grid(c.n_kv_heads, ((rows + 31) / 32 * G + 3) / 4, splits);
    if (D == 64) hipLaunchKernelGGL(attn_prefill_kernel<64>, grid, dim3(256), 0, st, a);
    else if (D == 128) hipLaunchKernelGGL(attn_prefill_kernel<128>, grid, dim3(256), 0, st, a);
    else return hipErrorInvalidValue;
    if (hipError_t e = hipGetLastError()) return e;
    return splits > 1 ? launch_combine(c, nullptr, splits, partial, rows, nullptr, out_tiled, nullptr, st) : hipSuccess;
}

}  // namespace sun
