// Small kernels of the decode step (Eq. 3): embedding gather, residual + RMSNorm,
// rotary embedding + KV append (Eq. 4), greedy argmax, and the
// layout helpers around the projection kernels.
#include "kernels.hpp"
#include "rows.hpp"

namespace sun {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void embed_rope_kernel(EmbedRope e) { embed_rope_row(e, blockIdx.x); }

// Writes eight consecutive values of row b (unit u = k / 8) into the fixed-point tile of a 4-bit projection.
// The 16 lanes that hold one 128-wide group share its scale (largest magnitude over the group); the first of
// them stores the scale and the sum of the group's integers.  Every lane of the wave must call it.
__device__ __forceinline__ void qtile_group16(uint8_t* tile, float2* qscale, ATile t, int b, int u, bool live,
                                              const float (&y)[8]) {
    float am = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) am = fmaxf(am, fabsf(y[e]));
    am = fmaxf(am, lane_xor<1>(am));
    am = fmaxf(am, lane_xor<2>(am));
    am = fmaxf(am, lane_xor<4>(am));
    am = fmaxf(am, lane_xor<8>(am));
    int sum = live ? qtile_store8(tile, t, b, u, y, qtile_inv(am)) : 0;
    sum += lane_xor<1>(sum);
    sum += lane_xor<2>(sum);
    sum += lane_xor<4>(sum);
    sum += lane_xor<8>(sum);
    if (live && (threadIdx.x & 15) == 0) qscale[(size_t)(u >> 4) * (t.MB * 32) + b] = float2{am / kQMax, __int_as_float(sum)};
}

// ---------------- residual add + RMSNorm ----------------
// One block per row.  x += sum_s partial[s] (s ascending), h = x * rsqrt(mean(x^2) + eps) * g.
struct NormArgs {
    float* x;
    const float* partial;
    const void* gain;
    float* h_f32;    // F32 only: row-major
    uint16_t* h_tiled;
    float2* qscale;  // not NULL: h_tiled is the fixed-point tile of a 4-bit projection, and this its scales and sums
    const uint32_t* lost;
    int nparts, ld_rows, H, mb;
    float eps;
};

// One 8-element unit per thread and pass (up to two passes, i.e. hidden <= 16 * blockDim), all
// slab loads of a unit independent of one another so that they are in flight together.
// LOST: behind the launch of all layers, which may have been given up.
template <bool F32, bool LOST>
__global__ __launch_bounds__(1024) void residual_norm_kernel(NormArgs a) {
    __shared__ float red[16];
    const int b = blockIdx.x, tid = threadIdx.x, H = a.H, nunits = H / 8, nthreads = blockDim.x;
    uint32_t lost = 0u;
    if constexpr (LOST) lost = *a.lost;
    float* xr = a.x + (size_t)b * H;
    float v[2][8];
    float ss = 0.f;
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const int u = tid + it * nthreads;
        if (u < nunits) {
            f32x4 lo = *reinterpret_cast<const f32x4*>(xr + u * 8), hi = *reinterpret_cast<const f32x4*>(xr + u * 8 + 4);
            const float* p = a.partial + (size_t)b * H + u * 8;
            const size_t slab = (size_t)a.ld_rows * H;
            for (int s0 = 0; s0 < a.nparts; s0 += 4) {
                f32x4 pl[4], ph[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int s = min(s0 + j, a.nparts - 1);
                    pl[j] = *reinterpret_cast<const f32x4*>(p + s * slab);
                    ph[j] = *reinterpret_cast<const f32x4*>(p + s * slab + 4);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (s0 + j < a.nparts) {  // slabs are added in ascending order
                        lo += pl[j];
                        hi += ph[j];
                    }
            }
            if (a.nparts > 0) {
                *reinterpret_cast<f32x4*>(xr + u * 8) = lo;
                *reinterpret_cast<f32x4*>(xr + u * 8 + 4) = hi;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[it][e] = lo[e];
                v[it][4 + e] = hi[e];
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) ss = fmaf(v[it][e], v[it][e], ss);
        }
    }
    ss = wave_sum(ss);
    if ((tid & 63) == 0) red[tid >> 6] = ss;
    __syncthreads();
    float tot = 0.f;
    for (int w = 0; w < nthreads / 64; ++w) tot += red[w];
    const float rinv = lost ? NAN : 1.0f / sqrtf(tot / (float)H + a.eps);
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const int u = tid + it * nthreads;
        float y[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (u < nunits) {
            float g[8];
            if constexpr (F32) {
#pragma unroll
                for (int e = 0; e < 8; ++e) g[e] = ((const float*)a.gain)[u * 8 + e];
            } else {
                const u32x4 gw = *reinterpret_cast<const u32x4*>((const uint16_t*)a.gain + u * 8);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    g[2 * e] = bf16_lo(gw[e]);
                    g[2 * e + 1] = bf16_hi(gw[e]);
                }
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] = v[it][e] * rinv * g[e];
            if constexpr (F32) {
                *reinterpret_cast<f32x4*>(a.h_f32 + (size_t)b * H + u * 8) = f32x4{y[0], y[1], y[2], y[3]};
                *reinterpret_cast<f32x4*>(a.h_f32 + (size_t)b * H + u * 8 + 4) = f32x4{y[4], y[5], y[6], y[7]};
            } else if (!a.qscale) {
                u32x4 o, ol;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    o[e] = pack_bf16(y[2 * e], y[2 * e + 1]);
                    ol[e] = pack_bf16(y[2 * e] - bf16_lo(o[e]), y[2 * e + 1] - bf16_hi(o[e]));
                }
                reinterpret_cast<u32x4*>(a.h_tiled)[atile_unit(ATile{a.mb}, 0, b, u)] = o;
                reinterpret_cast<u32x4*>(a.h_tiled)[atile_unit(ATile{a.mb}, 1, b, u)] = ol;
            }
        }
        if (!F32 && a.qscale)  // fixed-point tile of a 4-bit projection: 16 consecutive units (lanes) form one 128-wide group
            qtile_group16((uint8_t*)a.h_tiled, a.qscale, ATile{a.mb}, b, u, u < nunits, y);
    }
}

hipError_t launch_residual_norm(const sun_model_cfg& cfg, float* x, const float* partial, int nparts, int ld_rows,
                                const void* gain, int batch, float* h_f32, void* h_tiled, float* qscale, hipStream_t st, const uint32_t* lost) {
    NormArgs a{};
    a.x = x;
    a.partial = partial;
    a.gain = gain;
    a.h_f32 = h_f32;
    a.h_tiled = (uint16_t*)h_tiled;
    a.qscale = (float2*)qscale;
    a.lost = lost;
    a.nparts = nparts;
    a.ld_rows = ld_rows;
    a.H = cfg.hidden;
    a.mb = atile_for_rows(batch).MB;
    a.eps = cfg.rms_eps;
    if (cfg.hidden % 8 || cfg.hidden > 16 * 1024) return hipErrorInvalidValue;
    const int units = cfg.hidden / 8;
    const int threads = units <= 1024 ? (units + 63) / 64 * 64 : ((units + 1) / 2 + 63) / 64 * 64;
    if (h_f32) hipLaunchKernelGGL((residual_norm_kernel<true, false>), dim3(batch), dim3(threads), 0, st, a);
    else if (lost) hipLaunchKernelGGL((residual_norm_kernel<false, true>), dim3(batch), dim3(threads), 0, st, a);
    else hipLaunchKernelGGL((residual_norm_kernel<false, false>), dim3(batch), dim3(threads), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_embed_rope(const sun_model_cfg& cfg, const void* embed, const int32_t* tokens, const int32_t* seq_lens,
                             int first_pos, int rows, float* x, float* table, hipStream_t st) {
    hipLaunchKernelGGL(embed_rope_kernel, dim3(rows), dim3(256), 0, st, make_embed_rope(cfg, embed, tokens, seq_lens, first_pos, x, table));
    return hipGetLastError();
}

// ---------------- rotary embedding + KV append ----------------
// grid (Hq + 2*Hkv, batch): head index < Hq -> q head; next Hkv -> k head; last Hkv -> v head.
struct RopeArgs {
    const float* qkv;
    const float* table;
    const int32_t* seq_lens;
    const int32_t* page_tables;
    float* q_out;
    uint16_t* pool;
    int64_t k_base, k_page, k_head, k_token, k_dim, v_base, v_page, v_head, v_token, v_dim;
    int nparts, ld_rows, Hq, Hkv, D, max_pages, n_pages, first_pos;
    const void* qn;  // head-norm gains [D] for q and k heads, or NULL (no head norm)
    const void* kn;
    const void *bq, *bk, *bv;  // projection biases [Hq*D], [Hkv*D], [Hkv*D] (element type as the gains), or NULL
    int gain_bf16;
    float eps;
};

__global__ __launch_bounds__(64) void rope_append_kernel(RopeArgs a) {
    const int b = blockIdx.y, hh = blockIdx.x, D = a.D, half = D / 2;
    const int Nqkv = (a.Hq + 2 * a.Hkv) * D;
    // lengths and page ids are validated on the host under SUN_VALIDATE; clamp so bad input cannot fault
    const int L = min(max(a.seq_lens ? a.seq_lens[b] : a.first_pos + b, 0), a.max_pages * kPageTokens - 1);
    const int32_t* pt = a.page_tables + (a.seq_lens ? (size_t)b * a.max_pages : 0);
    const int page = min(max(pt[L / kPageTokens], 0), a.n_pages - 1);
    const int slot = L % kPageTokens;
    const float* src = a.qkv + (size_t)b * Nqkv + (size_t)hh * D;
    const size_t pstride = (size_t)a.ld_rows * Nqkv;
    // head_dim <= 128: lane j owns elements j and j + D/2; lanes past D/2 carry zeros through the norm
    const int j = threadIdx.x;
    const bool act = j < half;
    float lo = 0.f, hi = 0.f;
    if (act) {
        for (int s = 0; s < a.nparts; ++s) {
            lo += src[s * pstride + j];
            hi += src[s * pstride + j + half];
        }
    }
    if (a.bq && act) {  // bias of this head's slice of the q, k or v projection
        const void* bias = hh < a.Hq ? a.bq : hh < a.Hq + a.Hkv ? a.bk : a.bv;
        const int h0 = (hh < a.Hq ? hh : hh < a.Hq + a.Hkv ? hh - a.Hq : hh - a.Hq - a.Hkv) * D;
        lo += a.gain_bf16 ? bf16_bits_to_f32(((const uint16_t*)bias)[h0 + j]) : ((const float*)bias)[h0 + j];
        hi += a.gain_bf16 ? bf16_bits_to_f32(((const uint16_t*)bias)[h0 + j + half]) : ((const float*)bias)[h0 + j + half];
    }
    if (a.qn && hh < a.Hq + a.Hkv) {  // RMSNorm over the head's D elements (uniform branch: all lanes take part)
        const float ss = wave_sum(lo * lo + hi * hi);
        const float r = 1.0f / sqrtf(ss / (float)D + a.eps);
        if (act) {
            const void* g = hh < a.Hq ? a.qn : a.kn;
            const float gl = a.gain_bf16 ? bf16_bits_to_f32(((const uint16_t*)g)[j]) : ((const float*)g)[j];
            const float gh = a.gain_bf16 ? bf16_bits_to_f32(((const uint16_t*)g)[j + half]) : ((const float*)g)[j + half];
            lo = lo * r * gl;
            hi = hi * r * gh;
        }
    }
    if (!act) return;
    if (hh < a.Hq + a.Hkv) {
        const float c = a.table[((size_t)b * half + j) * 2], sn = a.table[((size_t)b * half + j) * 2 + 1];
        const float rl = lo * c - hi * sn, rh = hi * c + lo * sn;
        lo = rl;
        hi = rh;
    }
    if (hh < a.Hq) {
        a.q_out[((size_t)b * a.Hq + hh) * D + j] = lo;
        a.q_out[((size_t)b * a.Hq + hh) * D + j + half] = hi;
    } else if (hh < a.Hq + a.Hkv) {
        uint16_t* kd = a.pool + a.k_base + (int64_t)page * a.k_page + (int64_t)(hh - a.Hq) * a.k_head + slot * a.k_token;
        kd[j * a.k_dim] = f32_to_bf16_bits(lo);
        kd[(j + half) * a.k_dim] = f32_to_bf16_bits(hi);
    } else {
        uint16_t* vd = a.pool + a.v_base + (int64_t)page * a.v_page + (int64_t)(hh - a.Hq - a.Hkv) * a.v_head + slot * a.v_token;
        vd[j * a.v_dim] = f32_to_bf16_bits(lo);
        vd[(j + half) * a.v_dim] = f32_to_bf16_bits(hi);
    }
}

hipError_t launch_rope_append(const KvPool& pool, int layer, const float* qkv, int nparts, int ld_rows,
                              const float* table, const int32_t* seq_lens, int first_pos, const int32_t* page_tables, int max_pages,
                              int batch, float* q_out, const void* q_norm, const void* k_norm, const void* bq, const void* bk,
                              const void* bv, hipStream_t st) {
    const sun_model_cfg& c = pool.cfg;
    if (c.head_dim > 128) return hipErrorInvalidValue;
    const sun_kv_layout& L = pool.lay;
    RopeArgs a{};
    a.qkv = qkv;
    a.table = table;
    a.seq_lens = seq_lens;
    a.first_pos = first_pos;
    a.page_tables = page_tables;
    a.q_out = q_out;
    a.pool = pool.base;
    a.k_base = L.k_off + (int64_t)layer * L.k_layer;
    a.k_page = L.k_page;
    a.k_head = L.k_head;
    a.k_token = L.k_token;
    a.k_dim = L.k_dim;
    a.v_base = L.v_off + (int64_t)layer * L.v_layer;
    a.v_page = L.v_page;
    a.v_head = L.v_head;
    a.v_token = L.v_token;
    a.v_dim = L.v_dim;
    a.nparts = nparts;
    a.ld_rows = ld_rows;
    a.Hq = c.n_q_heads;
    a.Hkv = c.n_kv_heads;
    a.D = c.head_dim;
    a.max_pages = max_pages;
    a.n_pages = (int)L.n_pages;
    a.qn = c.qk_norm ? q_norm : nullptr;
    a.kn = c.qk_norm ? k_norm : nullptr;
    a.gain_bf16 = c.act_dtype == SUN_BF16;
    a.eps = c.rms_eps;
    a.bq = c.qkv_bias ? bq : nullptr;
    a.bk = c.qkv_bias ? bk : nullptr;
    a.bv = c.qkv_bias ? bv : nullptr;
    if (c.qk_norm && (!q_norm || !k_norm)) return hipErrorInvalidValue;
    if (c.qkv_bias && (!bq || !bk || !bv)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(rope_append_kernel, dim3(c.n_q_heads + 2 * c.n_kv_heads, batch), dim3(64), 0, st, a);
    return hipGetLastError();
}

// ---------------- SwiGLU over the gate/up projection's partial sums ----------------
// part: [nparts][ld_rows][2*ffn] fp32 with the projection's column order (blocks of 16 gate
// columns followed by their 16 up columns).  Writes u = silu(sum g) * (sum u) [rows, ffn] as the down
// projection's input: two-plane tiled bf16, or (qscale given) the fixed-point tile of a 4-bit projection.
__global__ __launch_bounds__(256) void swiglu_tile_kernel(const float* __restrict__ part, int nparts, int ld_rows,
                                                          int ffn, int mb, u32x4* __restrict__ tiled,
                                                          float* __restrict__ qscale) {
    const int b = blockIdx.y, u = blockIdx.x * 256 + threadIdx.x;  // unit = 8 consecutive u columns
    float y[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (u < ffn / 8) {
        const int j = u * 8;
        const float* p = part + (size_t)b * 2 * ffn + (j >> 4) * 32 + (j & 15);
        const size_t slab = (size_t)ld_rows * 2 * ffn;
        f32x4 g0 = {0.f, 0.f, 0.f, 0.f}, g1 = g0, u0 = g0, u1 = g0;
        for (int s = 0; s < nparts; ++s) {  // slabs in ascending order
            g0 += *reinterpret_cast<const f32x4*>(p + s * slab);
            g1 += *reinterpret_cast<const f32x4*>(p + s * slab + 4);
            u0 += *reinterpret_cast<const f32x4*>(p + s * slab + 16);
            u1 += *reinterpret_cast<const f32x4*>(p + s * slab + 20);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            y[e] = g0[e] / (1.f + __expf(-g0[e])) * u0[e];
            y[4 + e] = g1[e] / (1.f + __expf(-g1[e])) * u1[e];
        }
        if (!qscale) {
            u32x4 o, ol;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                o[e] = pack_bf16(y[2 * e], y[2 * e + 1]);
                ol[e] = pack_bf16(y[2 * e] - bf16_lo(o[e]), y[2 * e + 1] - bf16_hi(o[e]));
            }
            tiled[atile_unit(ATile{mb}, 0, b, u)] = o;
            tiled[atile_unit(ATile{mb}, 1, b, u)] = ol;
        }
    }
    if (qscale) qtile_group16((uint8_t*)tiled, (float2*)qscale, ATile{mb}, b, u, u < ffn / 8, y);
}

hipError_t launch_swiglu_tile(const float* part, int nparts, int ld_rows, int rows, int ffn, void* tiled, float* qscale,
                              hipStream_t st) {
    if (ffn % 128) return hipErrorInvalidValue;
    const int mb = atile_for_rows(rows).MB;
    hipLaunchKernelGGL(swiglu_tile_kernel, dim3((ffn / 8 + 255) / 256, rows), dim3(256), 0, st, part, nparts, ld_rows, ffn,
                       mb, (u32x4*)tiled, qscale);
    return hipGetLastError();
}

// ---------------- greedy argmax, lowest index on ties ----------------
// kArgmaxParts slices of a row are searched by one workgroup each, then a wave per row picks among the slice winners; a
// row of at most kArgmaxOne logits is searched by one workgroup in one launch.  An element that is not greater than
// -infinity (NaN included) is never picked; a row without any other yields 0.
// Bound by the read of the logits: 16-byte loads, all of a thread's in flight together.  128 256 logits, 4-byte loads one
// after the other -> these: 1 row 16.0 -> 4.5 us, 256 rows 43.3 -> 22.0 (6.0 TB/s).
struct Best {
    float v;
    int i;
};
__device__ __forceinline__ void better(Best& a, float v, int i) {
    if (v > a.v || (v == a.v && i < a.i)) a = Best{v, i};
}
__device__ __forceinline__ Best wave_best(Best a) {
    const auto exchange = [&](auto o) {
        Best b = a;
        swap_rows<decltype(o)::value>(a.v, b.v);
        swap_rows<decltype(o)::value>(a.i, b.i);
        better(a, b.v, b.i);
    };
    exchange(std::integral_constant<int, 32>{});
    exchange(std::integral_constant<int, 16>{});
    better(a, lane_xor<8>(a.v), lane_xor<8>(a.i));
    better(a, lane_xor<4>(a.v), lane_xor<4>(a.i));
    better(a, lane_xor<2>(a.v), lane_xor<2>(a.i));
    better(a, lane_xor<1>(a.v), lane_xor<1>(a.i));
    return a;
}
// logits j0 .. j1 - 1 of a row by a workgroup of 256; the result is in thread 0
__device__ __forceinline__ Best block_best(const float* row, int j0, int j1, bool vec) {
    __shared__ Best waves[4];
    const int tid = threadIdx.x;
    Best b{-INFINITY, 0x7fffffff};
    int j = j0;
    if (vec) {  // j0 is a multiple of four and the row starts on 16 bytes
        const int n4 = (j1 - j0) / 4;
        const f32x4* p = reinterpret_cast<const f32x4*>(row + j0);
        for (int q0 = tid; q0 < n4; q0 += 1024) {
            f32x4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = p[min(q0 + u * 256, n4 - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e)  // past the end the last four again: an index that loses its ties
                    if (v[u][e] > b.v) b = Best{v[u][e], j0 + min(q0 + u * 256, n4 - 1) * 4 + e};
        }
        j = j0 + n4 * 4;
    }
    for (j += tid; j < j1; j += 256) {  // a thread meets its indices in ascending order
        const float v = row[j];
        if (v > b.v) b = Best{v, j};
    }
    b = wave_best(b);
    if ((tid & 63) == 0) waves[tid >> 6] = b;
    __syncthreads();
    if (tid == 0)
        for (int w = 1; w < 4; ++w) better(b, waves[w].v, waves[w].i);
    return b;
}

__global__ __launch_bounds__(256) void argmax_part_kernel(const float* __restrict__ logits, int V, int per, int vec,
                                                          float* __restrict__ pval, int32_t* __restrict__ pidx,
                                                          int32_t* __restrict__ next, const uint32_t* __restrict__ lost) {
    const int b = blockIdx.y, part = blockIdx.x;
    const Best r = block_best(logits + (size_t)b * V, min(V, part * per), min(V, (part + 1) * per), vec != 0);
    if (threadIdx.x != 0) return;
    if (next) {
        next[b] = lost && *lost ? -1 : r.i == 0x7fffffff ? 0 : r.i;
    } else {
        pval[(size_t)b * kArgmaxParts + part] = r.v;
        pidx[(size_t)b * kArgmaxParts + part] = r.i;
    }
}

__global__ __launch_bounds__(256) void argmax_pick_kernel(const float* __restrict__ pval, const int32_t* __restrict__ pidx,
                                                          int batch, int32_t* __restrict__ next, const uint32_t* __restrict__ lost) {
    static_assert(kArgmaxParts <= 64, "a lane per slice");
    const int b = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (b >= batch) return;
    Best r{-INFINITY, 0x7fffffff};
    if (lane < kArgmaxParts) r = Best{pval[(size_t)b * kArgmaxParts + lane], pidx[(size_t)b * kArgmaxParts + lane]};
    r = wave_best(r);
    if (lane == 0) next[b] = lost && *lost ? -1 : r.i == 0x7fffffff ? 0 : r.i;
}

hipError_t launch_argmax(const float* logits, int batch, int vocab, float* part_val, int32_t* part_idx, int32_t* next,
                         const uint32_t* lost, hipStream_t st) {
    const bool one = vocab <= kArgmaxOne;
    const int per = one ? vocab : ((vocab + kArgmaxParts - 1) / kArgmaxParts + 3) / 4 * 4;
    const int vec = (uintptr_t)logits % 16 == 0 && vocab % 4 == 0;
    hipLaunchKernelGGL(argmax_part_kernel, dim3(one ? 1 : kArgmaxParts, batch), dim3(256), 0, st, logits, vocab, per, vec, part_val,
                       part_idx, one ? next : nullptr, lost);
    if (!one) hipLaunchKernelGGL(argmax_pick_kernel, dim3((batch + 3) / 4), dim3(256), 0, st, part_val, part_idx, batch, next, lost);
    return hipGetLastError();
}

// ---------------- KV ingest: a contiguous cache into a request's pages ----------------
// One workgroup per (logical page, kv head, layer).  Source [layer][token][head][dim] bf16; token t is
// position first_pos + t.  K rows are copied 16 bytes at a time; V goes through an LDS tile because the
// pool keeps it transposed ([dim][token]).  Only the positions of the source are written, so a chunk can
// be appended to a partly filled page.  A page id outside the pool skips the page.
//
// Bound by HBM: every byte is read once and written once.  A source larger than what the L2s of the chip hold (32 MB) is read with
// streaming loads, and one larger than the memory-side cache (256 MB) is written past the caches as well.  Below that the source
// is often still in the memory-side cache, having just been received, and stores that stream cost more than they save.
// Plain / loads streamed / loads and stores streamed (us), a source that has just been written, then one that no cache holds,
// destination cold: 36 MB 16.3 / 15.4 / 17.8, 24.5 / 18.5 / 19.2; 134 MB 43.6 / 44.5 / 57.3, 76 / 55 / 54; 268 MB 100 / 83 / 97,
// 129 / 103 / 101; 537 MB (32 layers x 4096 tokens) 211 / 186 / 197, 235 / 209 / 196, and one such hand-over after the other
// 189 / - / 169 (6.4 TB/s read plus written).  Only where source and destination both are those of the call before does the
// plain one win (36 MB 18.8 / 20.9 / 20.5).  Up to 8.4 MB a launch and its latency, and what it leaves in the caches the next
// step reads: plain 7.4, streamed 7.6.  Two heads to a workgroup (a source run of 512 bytes a token) is slower, 175 us for the
// 537 MB: half the workgroups, each with twice the work around its one barrier.
constexpr size_t kIngestStreamBytes = 32u << 20;   // bytes of the source, above which its loads stream
constexpr size_t kIngestThroughBytes = 256u << 20; // and its stores

template <bool STREAM, typename T>
__device__ __forceinline__ T ingest_load(const T* p) {
    if constexpr (STREAM) return load_stream(p);
    else return *p;
}
template <bool STREAM, typename T>
__device__ __forceinline__ void ingest_store(T v, T* p) {
    if constexpr (STREAM) __builtin_nontemporal_store(v, p);
    else *p = v;
}

struct IngestArgs {
    uint16_t* kbase;  // pool base + k_off
    uint16_t* vbase;
    int64_t k_layer, k_page, k_head, v_layer, v_page, v_head;
    const uint16_t* k_src;
    const uint16_t* v_src;
    const int32_t* page_table;
    int n_tokens, first_pos, Hkv, D, n_pages;
};

template <bool LOADS, bool STORES>
__global__ __launch_bounds__(256) void kv_ingest_kernel(IngestArgs a) {
    __shared__ uint16_t tile[kPageTokens][128 + 8];
    const int lp = a.first_pos / kPageTokens + blockIdx.x, h = blockIdx.y, l = blockIdx.z, tid = threadIdx.x;
    const int page = a.page_table[lp];
    if (page < 0 || page >= a.n_pages) return;
    const int p0 = lp * kPageTokens;
    const int s_lo = max(a.first_pos - p0, 0), s_hi = min(a.first_pos + a.n_tokens - p0, kPageTokens);  // valid slots
    const int D = a.D, cpt = D / 8;                                                                    // 16-byte chunks per token
    uint16_t* kd = a.kbase + l * a.k_layer + page * a.k_page + h * a.k_head;
    uint16_t* vd = a.vbase + l * a.v_layer + page * a.v_page + h * a.v_head;
    for (int idx = tid; idx < kPageTokens * cpt; idx += 256) {
        const int s = idx / cpt, c = idx % cpt;
        if (s < s_lo || s >= s_hi) continue;
        const size_t so = (((size_t)l * a.n_tokens + (p0 + s - a.first_pos)) * a.Hkv + h) * D + c * 8;
        const u32x4 k = ingest_load<LOADS>(reinterpret_cast<const u32x4*>(a.k_src + so));
        const u32x4 v = ingest_load<LOADS>(reinterpret_cast<const u32x4*>(a.v_src + so));
        ingest_store<STORES>(k, reinterpret_cast<u32x4*>(kd + s * D + c * 8));
        *reinterpret_cast<u32x4*>(&tile[s][c * 8]) = v;
    }
    __syncthreads();
    // V^T: thread <-> (dim, half of the page's 16 slots)
    for (int idx = tid; idx < D * 2; idx += 256) {
        const int dim = idx >> 1, half = idx & 1, s0 = half * 8;
        if (s0 >= s_lo && s0 + 8 <= s_hi) {
            uint16_t e[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) e[j] = tile[s0 + j][dim];
            u32x4 o;
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] = (uint32_t)e[2 * j] | ((uint32_t)e[2 * j + 1] << 16);
            ingest_store<STORES>(o, reinterpret_cast<u32x4*>(vd + dim * kPageTokens + s0));
        } else {
            for (int j = 0; j < 8; ++j)
                if (s0 + j >= s_lo && s0 + j < s_hi) vd[dim * kPageTokens + s0 + j] = tile[s0 + j][dim];
        }
    }
}

hipError_t launch_kv_ingest(const KvPool& pool, const void* k_src, const void* v_src, int n_tokens, int first_pos,
                            const int32_t* page_table, hipStream_t st) {
    const sun_model_cfg& c = pool.cfg;
    const sun_kv_layout& L = pool.lay;
    if (L.k_dim != 1 || L.k_token != c.head_dim || L.v_token != 1 || L.v_dim != kPageTokens || c.head_dim > 128 ||
        c.head_dim % 8)
        return hipErrorInvalidValue;
    IngestArgs a{};
    a.kbase = pool.base + L.k_off;
    a.vbase = pool.base + L.v_off;
    a.k_layer = L.k_layer; a.k_page = L.k_page; a.k_head = L.k_head;
    a.v_layer = L.v_layer; a.v_page = L.v_page; a.v_head = L.v_head;
    a.k_src = (const uint16_t*)k_src;
    a.v_src = (const uint16_t*)v_src;
    a.page_table = page_table;
    a.n_tokens = n_tokens;
    a.first_pos = first_pos;
    a.Hkv = c.n_kv_heads;
    a.D = c.head_dim;
    a.n_pages = (int)L.n_pages;
    const int pages = (first_pos + n_tokens - 1) / kPageTokens - first_pos / kPageTokens + 1;
    const size_t bytes = (size_t)2 * c.n_layers * n_tokens * c.n_kv_heads * c.head_dim * 2;
    const dim3 grid(pages, c.n_kv_heads, c.n_layers);
    if (bytes > kIngestThroughBytes) hipLaunchKernelGGL((kv_ingest_kernel<true, true>), grid, dim3(256), 0, st, a);
    else if (bytes > kIngestStreamBytes) hipLaunchKernelGGL((kv_ingest_kernel<true, false>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((kv_ingest_kernel<false, false>), grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

// ---------------- per-row inputs of a prefill block ----------------
__global__ __launch_bounds__(256) void prefill_rows_kernel(const int32_t* __restrict__ page_table, int max_pages,
                                                           int first_pos, int model_id, int32_t* __restrict__ tables,
                                                           int32_t* __restrict__ lens, int32_t* __restrict__ ids) {
    const int r = blockIdx.x;
    for (int c = threadIdx.x; c < max_pages; c += 256) tables[(size_t)r * max_pages + c] = page_table[c];
    if (threadIdx.x == 0) {
        lens[r] = first_pos + r;
        ids[r] = model_id;
    }
}

hipError_t launch_prefill_rows(const int32_t* page_table, int max_pages, int first_pos, int model_id, int rows,
                               int32_t* tables, int32_t* lens, int32_t* ids, hipStream_t st) {
    hipLaunchKernelGGL(prefill_rows_kernel, dim3(rows), dim3(256), 0, st, page_table, max_pages, first_pos, model_id,
                       tables, lens, ids);
    return hipGetLastError();
}

// ---------------- bookkeeping between the steps of a run ----------------
// One workgroup.  Request b feeds its generated token back and grows by one position.  If that
// position opens a page its table does not have yet, it takes the next unused entry of the free
// list; requests are served in index order (an exclusive scan over the requests that need a page).
// A request that finds the list empty, or whose table is full, keeps its length and re-decodes the
// same position; status bit 0 / bit 1 records that.  A request that got no token (next < 0) stays as it is, bit 2.
__global__ __launch_bounds__(1024) void advance_kernel(const int32_t* __restrict__ next, int batch, int max_pages,
                                                       const int32_t* __restrict__ free_pages, int n_free,
                                                       int32_t* __restrict__ token_ids, int32_t* __restrict__ page_tables,
                                                       int32_t* __restrict__ seq_lens, int32_t* __restrict__ free_head,
                                                       int32_t* __restrict__ status, int clear_status) {
    __shared__ int scan[1024];
    const int t = threadIdx.x;
    if (clear_status && t == 0) *status = 0;  // ordered before the atomicOr below by the barriers in between
    int new_len = 0, slot_page = 0, wants = 0, full = 0;
    const int token = t < batch ? next[t] : -1;
    if (token >= 0) {
        token_ids[t] = token;
        new_len = seq_lens[t] + 1;
        slot_page = new_len / kPageTokens;
        full = slot_page >= max_pages;
        wants = !full && new_len % kPageTokens == 0 && page_tables[(size_t)t * max_pages + slot_page] < 0;
    }
    scan[t] = wants;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        const int v = t >= o ? scan[t - o] : 0;
        __syncthreads();
        scan[t] += v;
        __syncthreads();
    }
    const int head = *free_head;
    const int rank = scan[t] - wants;  // requests before this one that take a page
    int flags = 0;
    if (t < batch) {
        if (token < 0) {
            flags = 4;
        } else if (full) {
            flags = 2;
        } else if (wants && head + rank >= n_free) {
            flags = 1;
        } else {
            if (wants) page_tables[(size_t)t * max_pages + slot_page] = free_pages[head + rank];
            seq_lens[t] = new_len;
        }
    }
    if (flags) atomicOr(status, flags);
    __syncthreads();  // every thread has read *free_head
    if (t == 1023) *free_head = min(head + scan[1023], n_free);
}

hipError_t launch_advance(const int32_t* next, int batch, int max_pages, const int32_t* free_pages, int n_free,
                          int32_t* token_ids, int32_t* page_tables, int32_t* seq_lens, int32_t* free_head,
                          int32_t* status, bool clear_status, hipStream_t st) {
    if (batch > 1024) return hipErrorInvalidValue;
    hipLaunchKernelGGL(advance_kernel, dim3(1), dim3(1024), 0, st, next, batch, max_pages, free_pages, n_free, token_ids,
                       page_tables, seq_lens, free_head, status, clear_status ? 1 : 0);
    return hipGetLastError();
}

// ---------------- between two steps of a small fp32 run ----------------
// The tokens of the step before (launch_argmax), the bookkeeping (advance_kernel) and the rows of the next step
// (embed_rope_row) in one launch instead of three, whose work is a few KB each.  Bound by latency.  A workgroup per request finds its
// token and gathers its embedding; one more keeps the books, for which no token is needed, and then makes the rotary tables of
// the new positions (the frequencies while it waits for the lengths).  Tiny configuration, three launches -> this (us a step): 1 / 8 / 48 requests 64.9 / 68.7 /
// 94.9 -> 62.5 / 66.3 / 89.6, the run of 16 steps with 8 requests 1141 -> 1034 us; all of it in one workgroup: 63.6 / 66.6 / 97.3.
// A row is searched by one workgroup, so long ones stay with the launches that search them by sixteen: one request of 4096 / 16 384 / 32 768 /
// 65 536 / 131 072 logits 66.8 / 72.9 / 86.3 / 100.7 / 114.8 -> 61.5 / 68.6 / 81.8 / 100.8 / 121.6, hence kTurnVocab.
struct TurnArgs {
    EmbedRope e;                    // x, table
    const float* logits;
    const int32_t* free_pages;
    int32_t *next, *token_ids, *page_tables, *seq_lens, *free_head, *status;
    int batch, max_pages, n_free, clear_status, last;
};

__global__ __launch_bounds__(256) void run_turn_kernel(TurnArgs a) {
    __shared__ int len[kTurnRows], tok_of_row;
    __shared__ double theta[64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, V = a.e.V, half = a.e.d / 2;
    if ((int)blockIdx.x < a.batch) {
        const int b = blockIdx.x;
        const Best r = block_best(a.logits + (size_t)b * V, 0, V, (uintptr_t)a.logits % 16 == 0 && V % 4 == 0);
        if (tid == 0) {
            const int t = r.i == 0x7fffffff ? 0 : r.i;
            a.next[b] = t;
            a.token_ids[b] = t;
            tok_of_row = min(max(t, 0), V - 1);
        }
        __syncthreads();
        if (a.last) return;
        for (int j = tid; j < a.e.H; j += 256) a.e.x[(size_t)b * a.e.H + j] = ((const float*)a.e.E)[(size_t)tok_of_row * a.e.H + j];
        return;
    }
    if (wave == 1 && lane < half) theta[lane] = rope_theta(a.e, lane);
    if (wave == 0) {                                       // advance_kernel's rules
        int new_len = 0, old_len = 0, slot_page = 0, full = 0;
        bool wants = false;
        if (lane < a.batch) {
            old_len = a.seq_lens[lane];
            new_len = old_len + 1;
            slot_page = new_len / kPageTokens;
            full = slot_page >= a.max_pages;
            wants = !full && new_len % kPageTokens == 0 && a.page_tables[(size_t)lane * a.max_pages + slot_page] < 0;
        }
        const int head = *a.free_head;
        const unsigned long long all = __ballot(wants);
        const int rank = __popcll(all & ((1ull << lane) - 1));
        int flags = 0;
        if (lane < a.batch) {
            if (full) {
                flags = 2;
            } else if (wants && head + rank >= a.n_free) {
                flags = 1;
            } else {
                if (wants) a.page_tables[(size_t)lane * a.max_pages + slot_page] = a.free_pages[head + rank];
                a.seq_lens[lane] = new_len;
            }
            len[lane] = flags ? old_len : new_len;
        }
        const int bits = (__ballot(flags & 1) ? 1 : 0) | (__ballot(flags & 2) ? 2 : 0);
        if (lane == 0) {
            *a.status = (a.clear_status ? 0 : *a.status) | bits;
            *a.free_head = min(head + (int)__popcll(all), a.n_free);
        }
    }
    __syncthreads();
    if (a.last) return;
    for (int i = tid; i < a.batch * half; i += 256) {
        const float2 cs = rope_pair(theta[i % half], len[i / half]);
        a.e.table[2 * i] = cs.x;
        a.e.table[2 * i + 1] = cs.y;
    }
}

hipError_t launch_run_turn(const sun_model_cfg& cfg, const void* embed, const float* logits, int batch, int max_pages, const int32_t* free_pages, int n_free,
                           int32_t* next, int32_t* token_ids, int32_t* page_tables, int32_t* seq_lens, int32_t* free_head, int32_t* status,
                           bool clear_status, bool last, float* x, float* table, hipStream_t st) {
    if (batch > kTurnRows || cfg.act_dtype != SUN_F32 || cfg.head_dim > 128) return hipErrorInvalidValue;
    const TurnArgs a{make_embed_rope(cfg, embed, nullptr, nullptr, 0, x, table), logits, free_pages, next, token_ids, page_tables, seq_lens, free_head, status,
                     batch, max_pages, n_free, clear_status, last};
    hipLaunchKernelGGL(run_turn_kernel, dim3(batch + 1), dim3(256), 0, st, a);
    return hipGetLastError();
}

// ---------------- continuous batching: retire, advance, admit between two steps ----------------
// One workgroup of 1024 threads; thread t < slots owns row t, and all 16 waves share the walks over page-table
// rows (a wave per row, 64 columns per load), so that no thread walks a row alone.  All orders are row order
// (exclusive scans) and column order (ballots), so the result does not depend on scheduling.  The phases
// follow the declaration of sun_decode_serve.
constexpr int kServeThreads = 1024;
constexpr int kServeWaves = kServeThreads / 64;

// exclusive prefix sum over the workgroup in thread order; total = the sum over all threads
__device__ __forceinline__ int block_scan_excl(int v, int* sc, int& total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(inc, o);
        if (lane >= o) inc += u;
    }
    __syncthreads();  // sc may still be read from the previous scan
    if (lane == 63) sc[w] = inc;
    __syncthreads();
    int before = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < kServeWaves; ++i) {
        const int part = sc[i];
        before += i < w ? part : 0;
        tot += part;
    }
    total = tot;
    return before + inc - v;
}

// pages (entries >= 0) in one table row, counted by a whole wave; the same value in every lane
__device__ __forceinline__ int wave_count_row(const int32_t* row, int max_pages) {
    const int lane = threadIdx.x & 63;
    int n = 0;
    for (int c0 = 0; c0 < max_pages; c0 += 64) {
        const int c = c0 + lane;
        const bool have = c < max_pages && row[c] >= 0;
        n += __popcll(__ballot(have));
    }
    return n;
}

__global__ __launch_bounds__(kServeThreads) void serve_kernel(ServeArgs a, const int32_t* __restrict__ next,
                                                              int32_t* __restrict__ tokens_out,
                                                              int32_t* __restrict__ req_out, int do_reset, int do_advance) {
    __shared__ int sc[kServeWaves];
    __shared__ int held[256];  // pages per row, later pages per admission candidate
    __shared__ int roff[256];  // ring offset of a retiring row's first page, else -1
    __shared__ int act[256];   // what happens to a row's table: -1 nothing, -2 written as idle, q >= 0 copied from waiting q
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const bool row = t < a.slots;
    int whead = a.counters[0], head = a.counters[1], tail = a.counters[2];
    int32_t* tab = a.page_tables + (size_t)(row ? t : 0) * a.max_pages;
    int req = -1, left = 0, len = 0, status = 0, retired = 0, generated = 0;
    if (row && !do_reset) {
        req = a.slot_req[t];
        left = a.slot_left[t];
        len = a.seq_lens[t];
    }
    if (!do_reset)
        for (int r = wave; r < a.slots; r += kServeWaves) {
            const int n = wave_count_row(a.page_tables + (size_t)r * a.max_pages, a.max_pages);
            if (lane == 0) held[r] = n;
        }
    __syncthreads();
    int my_held = (row && !do_reset) ? held[t] : 0;
    bool occ = req >= 0;
    bool clear = row && do_reset;  // rows to be written as idle
    if (do_advance) {
        const int tok = row ? next[t] : 0;
        const bool lost = tok < 0;   // a step without a result: the rows stay as they are
        if (row) {
            tokens_out[t] = occ ? tok : -1;
            req_out[t] = lost ? -1 : req;
        }
        if (lost) status |= 4;
        bool fin = false;
        if (occ && !lost) {
            left -= 1;
            generated = 1;
            fin = left == 0 || tok == a.eos_id;
        }
        // retire: pages to the ring's tail, rows in order, columns in order
        int give_total;
        const int give = (occ && fin) ? my_held : 0;
        const int off = block_scan_excl(give, sc, give_total);
        if (t < 256) roff[t] = (occ && fin) ? off : -1;
        __syncthreads();
        for (int r = wave; r < a.slots; r += kServeWaves) {
            if (roff[r] < 0) continue;  // the same for the whole wave
            const int32_t* src = a.page_tables + (size_t)r * a.max_pages;
            int at = tail + roff[r];
            for (int c0 = 0; c0 < a.max_pages; c0 += 64) {
                const int c = c0 + lane;
                const int pg = c < a.max_pages ? src[c] : -1;
                const unsigned long long m = __ballot(pg >= 0);
                if (pg >= 0) a.ring[(unsigned)(at + __popcll(m & ((1ull << lane) - 1ull))) % (unsigned)a.ring_cap] = pg;
                at += __popcll(m);
            }
        }
        if (occ && fin) {
            retired = 1;
            clear = true;
        }
        tail += give_total;
        __syncthreads();  // the ring entries written above may be taken below
        // advance the others
        const bool cont = occ && !fin && !lost;
        const int new_len = len + 1, col = new_len / kPageTokens;
        const int wants = cont && col < a.max_pages && new_len % kPageTokens == 0 && tab[col] < 0;
        int want_total;
        const int rank = block_scan_excl(wants, sc, want_total);
        if (cont) {
            if (col >= a.max_pages) {
                status |= 2;
            } else if (wants && head + rank >= tail) {
                status |= 1;
            } else {
                if (wants) {
                    tab[col] = a.ring[(unsigned)(head + rank) % (unsigned)a.ring_cap];
                    my_held += 1;
                }
                len = new_len;
            }
            a.token_ids[t] = tok;
            a.slot_left[t] = left;
            a.seq_lens[t] = len;
        }
        head = min(head + want_total, tail);
        if (fin) occ = false;
    }
    if (do_reset) occ = false;
    if (clear) {
        a.token_ids[t] = 0;
        a.seq_lens[t] = 0;
        a.model_ids[t] = 0;
        a.slot_req[t] = -1;
        a.slot_left[t] = 0;
    }
    // admission
    int out_total, idle_total, need_total, ok_total;
    const int outst = occ ? max(0, (len + left - 1) / kPageTokens + 1 - my_held) : 0;
    block_scan_excl(outst, sc, out_total);
    const int avail = (tail - head) - out_total;
    const bool idle = row && !occ;
    const int idle_rank = block_scan_excl(idle ? 1 : 0, sc, idle_total);
    const int ncand = max(0, min(idle_total, a.n_wait - whead));
    for (int q = wave; q < ncand; q += kServeWaves) {  // the scans above separate this from the last use of held[]
        const int n = wave_count_row(a.w_tables + (size_t)(whead + q) * a.max_pages, a.max_pages);
        if (lane == 0) held[q] = n;
    }
    __syncthreads();
    auto cut_budget = [&](int q, bool& cut) {
        const int room = a.max_pages * kPageTokens - a.w_lens[q];
        const int b = a.w_budget[q];
        cut = b > room;
        return max(1, min(b, room));
    };
    int need = 0;
    if (t < ncand) {
        const int q = whead + t;
        bool cut;
        const int b = cut_budget(q, cut);
        need = max(0, (a.w_lens[q] + b - 1) / kPageTokens + 1 - held[t]);
    }
    const int before = block_scan_excl(need, sc, need_total);
    // candidate t is admitted if it and all before it fit (needs are >= 0, so the admitted ones are a prefix)
    const int ok = t < ncand && before + need <= avail;
    block_scan_excl(ok, sc, ok_total);
    int what = clear ? -2 : -1;
    if (idle && idle_rank < ok_total) {
        const int q = whead + idle_rank;
        bool cut;
        const int b = cut_budget(q, cut);
        if (cut) status |= 2;
        what = q;
        a.token_ids[t] = a.w_token[q];
        a.seq_lens[t] = a.w_lens[q];
        a.model_ids[t] = a.w_model[q];
        a.slot_req[t] = a.w_req[q];
        a.slot_left[t] = b;
    }
    if (t < 256) act[t] = what;
    __syncthreads();  // also: every read of the old tables (retirement, tab[col]) is behind us
    for (int r = wave; r < a.slots; r += kServeWaves) {
        const int w = act[r];
        if (w == -1) continue;
        int32_t* dst = a.page_tables + (size_t)r * a.max_pages;
        const int32_t* src = w >= 0 ? a.w_tables + (size_t)w * a.max_pages : nullptr;
        for (int c = lane; c < a.max_pages; c += 64) dst[c] = src ? src[c] : (c == 0 ? a.idle_page : -1);
    }
    int ret_total, gen_total;
    block_scan_excl(retired, sc, ret_total);
    block_scan_excl(generated, sc, gen_total);
    if (status) atomicOr(&a.counters[3], status);
    if (t == 0) {
        a.counters[0] = whead + ok_total;
        a.counters[1] = head;
        a.counters[2] = tail;
        a.counters[4] += ret_total;
        a.counters[5] += ok_total;
        a.counters[6] += gen_total;
        a.counters[7] += do_advance;
    }
}

hipError_t launch_serve(const ServeArgs& a, const int32_t* next, int32_t* tokens_out, int32_t* req_out, bool reset,
                        bool advance, hipStream_t st) {
    if (a.slots < 1 || a.slots > 256) return hipErrorInvalidValue;
    hipLaunchKernelGGL(serve_kernel, dim3(1), dim3(kServeThreads), 0, st, a, next, tokens_out, req_out, reset ? 1 : 0,
                       advance ? 1 : 0);
    return hipGetLastError();
}

// ---------------- HBM read probe (measurement only) ----------------
// Reads `n_blocks` blocks of `block_units` 16-byte units each, in the order perm gives (or in address order),
// and does nothing with them but fold them into one word per thread: what a kernel that only streams from HBM
// reaches on this device, contiguous or in scattered blocks the size of one (page, head) K or V block.
template <int STREAM>
__global__ __launch_bounds__(256) void hbm_read_probe_kernel(const u32x4* __restrict__ src, long long n_blocks,
                                                             int block_units, const int32_t* __restrict__ perm,
                                                             uint32_t* __restrict__ sink) {
    auto ld = [](const u32x4* p) { return STREAM ? load_stream(p) : *p; };
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const long long gw = (long long)blockIdx.x * 4 + wave, nw = (long long)gridDim.x * 4;
    uint32_t acc = 0;
    for (long long b = gw; b < n_blocks; b += nw) {     // one block per wave and turn, four 16-byte loads per lane in flight
        const long long blk = perm ? perm[b] : b;
        const u32x4* p = src + blk * block_units;
        for (int u = lane; u < block_units; u += 256) {
            const u32x4 v0 = ld(p + u), v1 = ld(p + min(u + 64, block_units - 1)), v2 = ld(p + min(u + 128, block_units - 1)),
                        v3 = ld(p + min(u + 192, block_units - 1));
            acc ^= v0[0] ^ v0[3] ^ v1[1] ^ v1[2] ^ v2[0] ^ v2[2] ^ v3[1] ^ v3[3];
        }
    }
    sink[(size_t)blockIdx.x * 256 + threadIdx.x] = acc;
}

hipError_t launch_hbm_read_probe(const void* src, long long n_blocks, int block_units, const int32_t* perm, int grid,
                                 bool stream, uint32_t* sink, hipStream_t st) {
    if (stream) hipLaunchKernelGGL(hbm_read_probe_kernel<1>, dim3(grid), dim3(256), 0, st, (const u32x4*)src, n_blocks, block_units, perm, sink);
    else hipLaunchKernelGGL(hbm_read_probe_kernel<0>, dim3(grid), dim3(256), 0, st, (const u32x4*)src, n_blocks, block_units, perm, sink);
    return hipGetLastError();
}

// ---------------- layout helpers ----------------
__global__ __launch_bounds__(256) void tile_rows_kernel(const float* __restrict__ x, int rows, int K, int mb,
                                                        u32x4* __restrict__ tiled, float* __restrict__ qscale) {
    const int b = blockIdx.y;
    const int u = blockIdx.x * 256 + threadIdx.x;
    float y[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (u < K / 8) {
        const float* p = x + (size_t)b * K + u * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) y[e] = p[e];
        if (!qscale) {
            u32x4 o, ol;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                o[e] = pack_bf16(y[2 * e], y[2 * e + 1]);
                ol[e] = pack_bf16(y[2 * e] - bf16_lo(o[e]), y[2 * e + 1] - bf16_hi(o[e]));
            }
            tiled[atile_unit(ATile{mb}, 0, b, u)] = o;
            tiled[atile_unit(ATile{mb}, 1, b, u)] = ol;
        }
    }
    if (qscale) qtile_group16((uint8_t*)tiled, (float2*)qscale, ATile{mb}, b, u, u < K / 8, y);
}

hipError_t launch_tile_rows(const float* x, int rows, int K, void* tiled, float* qscale, hipStream_t st) {
    if (K % 128) return hipErrorInvalidValue;
    const int mb = atile_for_rows(rows).MB;
    hipLaunchKernelGGL(tile_rows_kernel, dim3((K / 8 + 255) / 256, rows), dim3(256), 0, st, x, rows, K, mb,
                       (u32x4*)tiled, qscale);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void reduce_partials_kernel(const float* __restrict__ partial, int nparts,
                                                              int ld_rows, int N, float* __restrict__ out) {
    const int b = blockIdx.y, n = blockIdx.x * 256 + threadIdx.x;
    if (n >= N) return;
    float v = 0.f;
    for (int s = 0; s < nparts; ++s) v += partial[((size_t)s * ld_rows + b) * N + n];
    out[(size_t)b * N + n] = v;
}

hipError_t launch_reduce_partials(const float* partial, int nparts, int ld_rows, int rows, int N, float* out,
                                  hipStream_t st) {
    hipLaunchKernelGGL(reduce_partials_kernel, dim3((N + 255) / 256, rows), dim3(256), 0, st, partial, nparts, ld_rows,
                       N, out);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void untile_rows_kernel(const uint16_t* __restrict__ tiled, int K, int mb,
                                                          float* __restrict__ out) {
    const int b = blockIdx.y, k = blockIdx.x * 256 + threadIdx.x;
    if (k >= K) return;
    out[(size_t)b * K + k] = bf16_bits_to_f32(tiled[atile_elem(ATile{mb}, 0, b, k)]) +
                             bf16_bits_to_f32(tiled[atile_elem(ATile{mb}, 1, b, k)]);
}

hipError_t launch_untile_rows(const void* tiled, int rows, int K, float* out, hipStream_t st) {
    const int mb = atile_for_rows(rows).MB;
    hipLaunchKernelGGL(untile_rows_kernel, dim3((K + 255) / 256, rows), dim3(256), 0, st, (const uint16_t*)tiled, K, mb,
                       out);
    return hipGetLastError();
}

}  // namespace sun
