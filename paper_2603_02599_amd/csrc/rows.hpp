// Per-row device code that more than one translation unit launches: embedding gather and rotary table.
#pragma once
#include "common.hpp"

namespace sun {

// theta_j = base^(-2j/d); with the wavelength-dependent scaling rule of the LLaMA-3.1 class (scaling = 1) it
// is kept, divided by `factor`, or blended between the two, depending on where 2*pi/theta_j lies relative to
// orig/high_freq and orig/low_freq.
struct RopeScale {
    int scaling, orig_max;
    double factor, low_freq, high_freq;
};

struct EmbedRope {
    const void* E;
    const int32_t* tokens;
    const int32_t* seq_lens;  // position of row b, or NULL: first_pos + b
    float* x;                 // [rows, H]
    float* table;             // [rows, d/2] pairs (cos, sin) of pos * theta_j, angle in double
    int is_bf16, vec, H, V, d, first_pos;
    double base;
    RopeScale rs;
};

inline EmbedRope make_embed_rope(const sun_model_cfg& cfg, const void* embed, const int32_t* tokens, const int32_t* seq_lens,
                                 int first_pos, float* x, float* table) {
    const bool bf = cfg.act_dtype == SUN_BF16;
    return EmbedRope{embed, tokens, seq_lens, x, table, bf, bf && (uintptr_t)embed % 16 == 0 && cfg.hidden % 8 == 0, cfg.hidden,
                     cfg.vocab, cfg.head_dim, first_pos, (double)cfg.rope_base,
                     RopeScale{cfg.rope_scaling, cfg.rope_original_max_position, (double)cfg.rope_factor,
                               (double)cfg.rope_low_freq_factor, (double)cfg.rope_high_freq_factor}};
}

__device__ __forceinline__ double rope_theta(const EmbedRope& e, int j) {
    double theta = pow(e.base, -2.0 * (double)j / (double)e.d);
    if (e.rs.scaling == 1) {
        const double wavelen = 2.0 * 3.14159265358979323846 / theta, orig = (double)e.rs.orig_max;
        if (wavelen > orig / e.rs.low_freq) {
            theta = theta / e.rs.factor;
        } else if (wavelen >= orig / e.rs.high_freq) {
            const double smooth = (orig / wavelen - e.rs.low_freq) / (e.rs.high_freq - e.rs.low_freq);
            theta = (1.0 - smooth) * theta / e.rs.factor + smooth * theta;
        }
    }
    return theta;
}
// cosine and sine of position * theta
__device__ __forceinline__ float2 rope_pair(double theta, int position) {
    const double ang = (double)position * theta;
    return float2{(float)cos(ang), (float)sin(ang)};
}

// x[b] = E[token_b], and row b's cosines and sines; a workgroup of 256
__device__ __forceinline__ void embed_rope_row(const EmbedRope& e, int b) {
    const int tid = threadIdx.x;
    if (tid < e.d / 2) {
        const float2 cs = rope_pair(rope_theta(e, tid), e.seq_lens ? e.seq_lens[b] : e.first_pos + b);
        e.table[((size_t)b * (e.d / 2) + tid) * 2] = cs.x;
        e.table[((size_t)b * (e.d / 2) + tid) * 2 + 1] = cs.y;
    }
    const int tok = min(max(e.tokens[b], 0), e.V - 1);  // ids are validated on the host under SUN_VALIDATE; never fault here
    float* x = e.x + (size_t)b * e.H;
    if (e.vec) {  // bf16 rows that start on 16 bytes
        const u32x4_s* src = reinterpret_cast<const u32x4_s*>((const uint16_t*)e.E + (size_t)tok * e.H);
        for (int u = tid; u < e.H / 8; u += 256) {
            const u32x4_s w = src[u];
            *reinterpret_cast<f32x4*>(x + u * 8) = f32x4{bf16_lo(w[0]), bf16_hi(w[0]), bf16_lo(w[1]), bf16_hi(w[1])};
            *reinterpret_cast<f32x4*>(x + u * 8 + 4) = f32x4{bf16_lo(w[2]), bf16_hi(w[2]), bf16_lo(w[3]), bf16_hi(w[3])};
        }
        return;
    }
    for (int j = tid; j < e.H; j += 256)
        x[j] = e.is_bf16 ? bf16_bits_to_f32(((const uint16_t*)e.E)[(size_t)tok * e.H + j]) : ((const float*)e.E)[(size_t)tok * e.H + j];
}

}  // namespace sun
