// Shared device/host helpers of the SUN shared-decode library (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <vector>

#include "../../include/sun.h"

namespace sun {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

constexpr int kWave = 64;
constexpr int kPageTokens = 16;     // tokens per KV page
constexpr int kAttnChunk = 256;  // tokens per full split-K work item
constexpr int kAttnSmall = 64;   // tokens per small work item at the end of a request
// Length of a request's full chunks.  From 64 requests up it is kAttnChunk.  A smaller batch has too few
// chunks of that length to occupy the chip (and one wave walks a chunk step by step, a memory latency per
// step), so there the length is the power of two in [kAttnSmall, kAttnChunk] that gives about 2048 items over
// the whole batch if every request were like this one.  It depends on the request's own length, the batch
// size and the number of KV heads, never on the other requests, so a request's result does not depend on its
// batch-mates.
__host__ __device__ inline int attn_full_chunk(int n, int batch, int Hkv) {
    if (batch >= 64) return kAttnChunk;
    const long long target = (long long)n * Hkv * batch / 2048;
    int ch = kAttnSmall;
    while (2 * ch <= target && 2 * ch <= kAttnChunk) ch *= 2;
    return ch;
}
// All but the last full chunk's worth of tokens go into full chunks of length ch, the remaining
// 1 .. 2*ch-1 tokens into small chunks.
__host__ __device__ inline void attn_chunking(int n, int batch, int Hkv, int& n_full, int& n_small, int& ch) {
    ch = attn_full_chunk(n, batch, Hkv);
    const int f = n / ch;
    n_full = f > 1 ? f - 1 : 0;
    n_small = (n - n_full * ch + kAttnSmall - 1) / kAttnSmall;
}
constexpr int kGroup = 128;         // quantisation group along K (Appendix A.1)
constexpr int kMaxGroup = 8;        // query heads per KV head
constexpr int kMaxBatchTile = 256;  // rows of a decode batch
constexpr int kMaxPrefillTile = 2048;  // rows of a prefill block (bf16 projections only)

// ---- bf16 <-> f32 (round to nearest even, by the hardware's converter: one instruction for two values) ----
// The bits of every value are those of rounding by hand (all 2^32 compared; a NaN stays one but keeps its sign and payload's upper bits),
// which took six instructions a value in the kernels' tails: 8 layers of the 8B shape at 16 / 150 (4-bit) requests 1181 / 3068 ->
// 1165 / 3048 us, 5 requests 4-bit 678 -> 667, prefill of 1024 tokens 6528 -> 6461.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ float bf16_bits_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{lo, hi}, bf16x2_t));
}

// ---- projection activations: "fragment-tiled" two-plane bf16 layout ----
// An fp32 activation x is carried into the matrix cores as two bf16 values, hi = bf16(x) and
// lo = bf16(x - hi) (16 significant bits together); the projection multiplies both planes with
// the same weight fragment and adds the two results.  Rounding activations to a single bf16
// would make the result depend on which way values near a rounding boundary fall, and a deep
// stack amplifies that noise beyond the parity tolerance.
// A [rows, K] is stored so that one staging step of the MFMA projection kernels is a linear
// copy into LDS and each 16-byte unit (8 consecutive k of one row) is one lane's A operand of a
// 32x32x16 MFMA.  With MB = number of 32-row blocks of real rows (1, 2, 4 or a multiple of 8) the tiling has
// 2*MB blocks, plane p of row block r at block p*MB + r:
//   unit(p, b, k/8) = ((chunk * 8 + kk) * 2*MB + p*MB + b/32) * 64 + half * 32 + b%32
// with chunk = k / 128, g = (k % 128) / 8, half = g / 8, kk = g % 8.  Lane-half `half` of k-step
// kk of a 128-wide chunk therefore carries k = chunk*128 + half*64 + kk*8 .. +7; the packed
// weights use the same assignment, and any bijection is valid because the MFMA sums over k.
struct ATile {
    int MB;
};
__host__ __device__ __forceinline__ ATile atile_for_rows(int rows) {
    return ATile{rows <= 32 ? 1 : rows <= 64 ? 2 : rows <= 128 ? 4 : (rows + 255) / 256 * 8};
}
__host__ __device__ __forceinline__ size_t atile_unit(ATile t, int plane, int b, int k8) {
    const int chunk = k8 >> 4, g = k8 & 15;
    const int half = g >> 3, kk = g & 7;
    return ((size_t)(chunk * 8 + kk) * (2 * t.MB) + plane * t.MB + (b >> 5)) * 64 + half * 32 + (b & 31);
}
__host__ __device__ __forceinline__ size_t atile_elem(ATile t, int plane, int b, int k) {
    return atile_unit(t, plane, b, k >> 3) * 8 + (k & 7);
}
__host__ __device__ __forceinline__ size_t atile_bytes(ATile t, int K) { return (size_t)2 * t.MB * 32 * K * 2; }
// hi/lo split of one value; returns hi bits, lo bits via reference
__device__ __forceinline__ uint16_t split_bf16(float x, uint16_t& lo) {
    const uint16_t hi = f32_to_bf16_bits(x);
    lo = f32_to_bf16_bits(x - bf16_bits_to_f32(hi));
    return hi;
}

// ---- 4-bit projections: activations as 16-bit fixed point in two int8 planes ----
// The 4-bit codes are integers, so the quantised projections run on the int8 matrix cores with exact
// int32 sums (Eq. 8 evaluated on the integer grid; the scales are applied to the sums in fp32).  Per row
// and 128-wide group (the weights' group) an activation is x ~ sx * xi with sx = max|x| / kQMax and the
// integer xi = 256 * hi + lo, hi and lo in [-128, 127]: 16 bits below the group's largest value.  The
// producer of the activations also stores sx and sum_k xi (for the zero point) per row and group.
// Tile: 16-byte units of 16 consecutive k of one row and plane, ordered [group][k-step 0..3][plane]
// [32-row block][lane = half * 32 + row % 32] with k = group * 128 + half * 64 + step * 16 + (0..15):
// a unit is one lane's operand of a 32x32x32 int8 MFMA.
constexpr float kQMax = 32639.f;  // 127 * 256 + 127
__host__ __device__ __forceinline__ size_t qtile_unit(ATile t, int plane, int b, int k16) {
    const int c = k16 >> 3, g = k16 & 7, half = g >> 2, s = g & 3;
    return ((size_t)((c * 4 + s) * 2 + plane) * t.MB + (b >> 5)) * 64 + half * 32 + (b & 31);
}
// eight consecutive values of one row (k8 = index of the octet) -> their bytes in both planes; returns sum of xi
__device__ __forceinline__ int qtile_store8(uint8_t* tile, ATile t, int b, int k8, const float (&x)[8], float inv) {
    uint32_t hi[2] = {0u, 0u}, lo[2] = {0u, 0u};
    int sum = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int xi = (int)rintf(x[e] * inv);
        const int l = ((xi + 128) & 255) - 128, h = (xi - l) >> 8;
        sum += xi;
        hi[e >> 2] |= (uint32_t)(h & 255) << (8 * (e & 3));
        lo[e >> 2] |= (uint32_t)(l & 255) << (8 * (e & 3));
    }
    *reinterpret_cast<uint2*>(tile + qtile_unit(t, 0, b, k8 >> 1) * 16 + (k8 & 1) * 8) = uint2{hi[0], hi[1]};
    *reinterpret_cast<uint2*>(tile + qtile_unit(t, 1, b, k8 >> 1) * 16 + (k8 & 1) * 8) = uint2{lo[0], lo[1]};
    return sum;
}
// 1 / sx for a group whose largest magnitude is amax (an all-zero group maps to zeros with sx = 0)
__device__ __forceinline__ float qtile_inv(float amax) { return amax > 0.f ? kQMax / amax : 0.f; }

// 16-byte load of data that is read once and never again by this launch (the cached K and V of the attention kernel):
// streamed past the caches (the "nt" form of the load), which also leaves what the neighbouring kernels exchange
// in place.  Pays where an instruction reads long contiguous runs; see the attention kernel.
typedef uint32_t u32x4_s __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x4_s load_stream(const u32x4_s* p) { return __builtin_nontemporal_load(p); }

// 16 bytes a lane from memory straight into LDS: lane i's, at base + lane_bytes, land at lds_byte + 16 i.  No register
// holds the data and the compiler does not know of the request: whoever reads the place waits for it by hand (vmcnt,
// then the workgroup's barrier).  base and lds_byte are the same for the whole wave.  base has to come out of scalar
// instructions: a scalar register that a vector instruction (a lane read, say) wrote may be read by a vector memory instruction
// five wait states later, which the compiler does not insert in front of assembly (the compiled kernels are checked for it by
// a test; a scalar copy here or longer waits cost 1 to 2 % of a 4-bit step of few requests).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // m0 is a reserved register: it is overwritten here, and nobody is promised its value
__device__ __forceinline__ void lds_dma16(const void* base, uint32_t lane_bytes, uint32_t lds_byte) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_byte), "v"(lane_bytes), "s"(base) : "memory", "m0");
}
// The same with 4 bytes a lane: lane i's land at lds_byte + 4 i.
__device__ __forceinline__ void lds_dma4(const void* base, uint32_t lane_bytes, uint32_t lds_byte) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds_byte), "v"(lane_bytes), "s"(base) : "memory", "m0");
}
#pragma clang diagnostic pop
// Read-only data of the launch at an address that is the same for the whole wave, through the scalar cache.
__device__ __forceinline__ int32_t load_uniform(const int32_t* p) {
    return *(const __attribute__((address_space(4))) int32_t*)(uintptr_t)p;
}

// ---- data that workgroups of one launch hand to one another ----
// Stores that go through to memory and loads that do not take what this XCD's caches hold (each of the eight XCDs has an L2 of
// its own).  A store has arrived when vmcnt says so; no cache has to be written back or invalidated as a whole.
__device__ __forceinline__ void st_agent(float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void st_agent(uint32_t* p, uint32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void st_agent(uint16_t* p, uint16_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float ld_agent(const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ uint32_t ld_agent(const uint32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// two floats, eight bytes aligned
__device__ __forceinline__ void st_agent2(float* p, float a, float b) {
    __hip_atomic_store((unsigned long long*)p, (unsigned long long)__float_as_uint(a) | (unsigned long long)__float_as_uint(b) << 32,
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 ld_agent2(const float* p) {
    const unsigned long long v = __hip_atomic_load((const unsigned long long*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return float2{__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32))};
}

// ---- lanes of a wave reading one another ----
// The vector ALU moves a value within a row of 16 lanes while it computes (DPP) and exchanges rows in one instruction, some 10
// cycles a step where a shuffle through LDS takes 60 to 100; an all-lane sum is six steps in a row and ends most of the step's small
// kernels.  Against shuffles, the same bits: tiny fp32 run of 16 steps 1034 -> 967 us, 8 layers of the 8B shape, 4 bits, 5 requests 735 -> 726,
// 32 layers at 64 requests 8076 -> 8008.  All lanes have to be active.
template <int CTRL, class T>
__device__ __forceinline__ T lane_dpp(T v) {
    static_assert(sizeof(T) == 4, "a register");
    return __builtin_bit_cast(T, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
// the 16-lane rows (O = 16) or 32-lane halves (O = 32) of a and b with the odd ones of a and the even ones of b exchanged
template <int O, class T>
__device__ __forceinline__ void swap_rows(T& a, T& b) {
    static_assert(sizeof(T) == 4 && (O == 16 || O == 32), "");
    uint32_t x = __builtin_bit_cast(uint32_t, a), y = __builtin_bit_cast(uint32_t, b);
    if constexpr (O == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
        x = r[0];
        y = r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
        x = r[0];
        y = r[1];
    }
    a = __builtin_bit_cast(T, x);
    b = __builtin_bit_cast(T, y);
}
// lane l gets lane l ^ O's
template <int O, class T>
__device__ __forceinline__ T lane_xor(T v) {
    if constexpr (O == 1) return lane_dpp<0xB1>(v);                       // lanes 1 0 3 2 of every four
    else if constexpr (O == 2) return lane_dpp<0x4E>(v);                  // lanes 2 3 0 1
    else if constexpr (O == 4) return lane_dpp<0x1B>(lane_dpp<0x141>(v)); // l ^ 7 of every eight, then l ^ 3
    else if constexpr (O == 8) return lane_dpp<0x128>(v);                 // rotated by eight of sixteen
    else {
        T a = v, b = v;
        swap_rows<O>(a, b);
        return threadIdx.x & O ? a : b;
    }
}
// f over all lanes, in the order of a butterfly over lane bits 5 .. 0 (fixed => deterministic); f commutes.  Behind the step
// over bit 3 a row repeats after eight lanes, so a rotation by four reads what lane l ^ 4 holds, and so on.
template <class T, class F>
__device__ __forceinline__ T wave_all(T v, F f) {
    T a = v, b = v;
    swap_rows<32>(a, b);
    v = f(a, b);
    a = b = v;
    swap_rows<16>(a, b);
    v = f(a, b);
    v = f(v, lane_dpp<0x128>(v));
    v = f(v, lane_dpp<0x124>(v));
    v = f(v, lane_dpp<0x122>(v));
    return f(v, lane_dpp<0x121>(v));
}
__device__ __forceinline__ float wave_sum(float v) {
    return wave_all(v, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ int wave_sum(int v) {
    return wave_all(v, [](int a, int b) { return a + b; });
}
__device__ __forceinline__ float wave_max(float v) {
    return wave_all(v, [](float a, float b) { return fmaxf(a, b); });
}

// Maxima over eight lanes at a time and up to there: a lane gets the largest of `start` and all m up to the end of its eight lanes;
// before, the same up to their start.
__device__ __forceinline__ float wave_octet_max(float m, float start, float& before) {
    const auto moved = [](float old, float v, auto ctrl, auto rows, auto banks) {   // lanes that nothing moves to keep old
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old), __builtin_bit_cast(int, v), decltype(ctrl)::value,
                                                                     decltype(rows)::value, decltype(banks)::value, false));
    };
    typedef std::integral_constant<int, 0x118> Right8;    // within a row of 16 lanes
    typedef std::integral_constant<int, 0x142> NextRow;   // a row's last lane to the row behind it
    typedef std::integral_constant<int, 0x143> UpperHalf; // lane 31 to rows 2 and 3
    typedef std::integral_constant<int, 0xf> All;
    const float none = -INFINITY;
    float top = fmaxf(m, lane_xor<1>(m));
    top = fmaxf(top, lane_xor<2>(top));
    top = fmaxf(top, lane_dpp<0x141>(top));               // mirrored within eight lanes: the other four
    top = fmaxf(top, moved(none, top, Right8{}, All{}, All{}));
    top = fmaxf(top, moved(none, top, NextRow{}, std::integral_constant<int, 0xa>{}, All{}));
    top = fmaxf(top, moved(none, top, UpperHalf{}, std::integral_constant<int, 0xc>{}, All{}));
    top = fmaxf(top, start);
    before = moved(start, top, NextRow{}, std::integral_constant<int, 0xe>{}, std::integral_constant<int, 0x3>{});
    before = moved(before, top, Right8{}, All{}, std::integral_constant<int, 0xc>{});
    return top;
}

// Packed weights of a model from which they are streamed past the caches: the memory-side cache's 256 MB, in which those of a
// smaller model stay from one step to the next.
constexpr size_t kStreamWeightBytes = (size_t)256 << 20;

// ---- handles ----
struct KvPool {
    sun_model_cfg cfg;
    uint16_t* base;
    sun_kv_layout lay;
    int n_source_models;
    std::vector<int64_t> ingested;  // tokens ingested per source model (host side)
};

enum MatKind { MAT_NONE = 0, MAT_F32 = 1, MAT_BF16_PACKED = 2, MAT_W4_PACKED = 3, MAT_W4_LOGICAL = 4 };

// One projection matrix as the kernels consume it.
struct Mat {
    int kind = MAT_NONE;
    int N = 0, K = 0;          // logical out/in features (N counts gate+up rows for the fused pair)
    const void* w = nullptr;   // F32: row-major fp32; BF16_PACKED / W4_PACKED: packed codes
    const void* sz = nullptr;  // W4_PACKED: half2 (scale, zero) per (32-row block, group, row); or, with
                               // s_only, the fp16 scales alone, two groups per dword (zero point 8 everywhere)
    bool s_only = false;
    bool stream = false;       // BF16_PACKED: the model's weights together exceed kStreamWeightBytes
    bool vocab = false;        // the vocabulary projection
    // W4_LOGICAL (fp32 activations): logical arrays, up to two stacked sources (gate, up)
    const uint8_t* q[3] = {nullptr, nullptr, nullptr};
    const uint16_t* s[3] = {nullptr, nullptr, nullptr};
    const uint16_t* z[3] = {nullptr, nullptr, nullptr};
    const void* wsrc[3] = {nullptr, nullptr, nullptr};  // F32: separate row-major sources
    int nsrc = 0;
    int src_rows[3] = {0, 0, 0};
};

struct LayerW {
    const void* g1;
    const void* g2;
    const void* qn = nullptr;  // head-norm gains [head_dim], only with cfg.qk_norm
    const void* kn = nullptr;
    const void *bq = nullptr, *bk = nullptr, *bv = nullptr;  // projection biases, only with cfg.qkv_bias
    Mat qkv, o, gu, down;
};

struct Weights {
    sun_model_cfg cfg;
    bool quant;
    size_t packed;   // bytes of the packed matrices
    const void* embed;
    const void* gf;
    Mat lm;
    LayerW* layers;
};

void set_error(const char* fmt, ...);

}  // namespace sun

#define SUN_HIP_CHECK(expr)                                                              \
    do {                                                                                 \
        hipError_t e_ = (expr);                                                          \
        if (e_ != hipSuccess) {                                                          \
            sun::set_error("%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_), __FILE__, __LINE__); \
            return SUN_ERR_HIP;                                                          \
        }                                                                                \
    } while (0)
