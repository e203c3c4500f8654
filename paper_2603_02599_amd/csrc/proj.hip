// Projections of the decode step: out[b, n] = sum_k W[n, k] x[b, k] for the skinny
// batch (b <= 256) against the shared decode weights (Section 3.1, Eq. 3), and the
// QSUN variant with W_hat = (Q - Z) * S, 4-bit codes in groups of 128 along k
// (Section 3.3, Eq. 8; Appendix A.1).
//
// bf16 path: each weight byte is read from HBM once.  Weights are pre-tiled so that a
// wave's 16-byte-per-lane load is 1 KiB contiguous and already is the B operand of a
// 32x32x16 MFMA (lane n%32 <-> weight row, lane half <-> k octet).  Activations are
// pre-tiled by their producer, staged through LDS (double buffered) and shared by the
// waves of a workgroup; wave w owns 32 output columns and all batch rows.
//
// W4 path (proj_w4_kernel): the codes stay integers.  Activations arrive as 16-bit fixed point in two
// int8 planes with one scale per row and group (see common.hpp), the 4-bit codes are widened to bytes
// (an and, a shift-and per four codes) and both go through the 32x32x32 int8 MFMA, whose int32 sums
// are exact.  Per 128-wide group:  acc += (S * sx) * (256 * sum_k q_k hi_k + sum_k q_k lo_k - Z * sum_k xi_k),
// which is sum_k (q_k - Z) S (sx xi_k) up to the rounding of one int -> fp32 conversion and one fma.
#include <hip/hip_fp16.h>

#include <type_traits>

#include "kernels.hpp"

namespace sun {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// One 16-byte piece of the weights.  A launch of one row tile (up to 64 rows) reads every piece once, 1 KiB contiguous
// per wave, and streams it past the caches where the whole model is larger than the memory-side cache (kStreamWeightBytes);
// several row tiles share their fetches through L2 and load plainly, and so does a model that stays in the cache from one
// step to the next.
// Measured, 8B shape, plain -> streamed (us): gate/up at 1 / 64 rows 45.1 -> 41.0 / 47.6 -> 44.8, lm_head at 1 row
// 193 -> 177, q/k/v and o unchanged (bound by the launch around them), and so are the 4-bit launches (a quarter of the bytes).
// Steps at 1 / 8 / 64 requests, hidden 1024, by the model's weights, plain against streamed (us): 146 MB 237 / 253 / 300
// against 252 / 266 / 314, 214 MB 370 / 398 / 477 against 387 / 420 / 485, 259 MB 476 / 515 / 603 against 486 / 506 / 599, 304 MB
// 605 / 640 / 722 against 581 / 622 / 710, 575 MB 1189 / 1266 / 1421 against 1108 / 1216 / 1393.
template <bool STREAM>
__device__ __forceinline__ u32x4 load_w16(const u32x4* p) {
    if constexpr (STREAM) return load_stream(p);
    else return *p;
}

struct ProjArgs {
    const u32x4* W;
    const uint32_t* SZ;
    int s_only;    // W4: SZ holds fp16 scales only, two 128-wide groups per dword; the zero point is 8 everywhere
    const u32x4* A;
    const float* qscale;
    float* out;
    int rows, N, K;
    int n_stages, stages_per_split;
    int ldo, ld_rows;
    int mb_rows;   // 32-row blocks of real rows in the activation tiling (it holds twice as many: hi and lo plane)
};

// SwiGLU of a strip's accumulators.  A strip's 32 columns are 16 gate columns followed by the 16 up columns of the same u
// columns (the packing order of the pair), so lane c and lane c + 16 hold gate and up of u column c for the same sixteen
// rows of a row block.  They share the work: of every pair of rows the gate lane finishes one and the up lane the
// other, one exchange per pair.  sw: this wave's scratch, [plane][32 row blocks' rows][16] bf16, rows rl0 + 0..31.
template <int ROWS>
__device__ __forceinline__ void swiglu_strip(const f32x16& acc, uint16_t* sw, int rl0) {
    const int lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
    const bool up_lane = col >= 16;
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
        const float got = lane_xor<16>(up_lane ? acc[r] : acc[r + 1]);
        const float g = up_lane ? got : acc[r], up = up_lane ? acc[r + 1] : got;
        const float y = g / (1.f + __expf(-g)) * up;
        const uint16_t hi = f32_to_bf16_bits(y);
        const uint16_t lo = f32_to_bf16_bits(y - bf16_bits_to_f32(hi));
        const int rl = rl0 + 8 * (r >> 2) + 4 * half + (r & 3) + (up_lane ? 1 : 0);
        sw[(0 * ROWS + rl) * 16 + (col & 15)] = hi;
        sw[(1 * ROWS + rl) * 16 + (col & 15)] = lo;
    }
}

// MB counts the 32-row operand blocks of the workgroup: MR = MB/2 blocks of rows, each present
// as a hi and a lo bf16 plane (operand block m < MR is the hi plane of row block m, block MR+m
// its lo plane); both are multiplied with the same weight fragment into the same accumulator.
template <int MB, int KS, int NW, int EPI, int NBUF, bool STREAM>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
void proj_kernel(ProjArgs a) {
    constexpr int MR = MB / 2;
    static_assert(MB % 2 == 0, "operand blocks come in hi/lo pairs");
    constexpr int KK = KS / 16;                // MFMA k-steps per stage
    constexpr int STAGE_UNITS = KK * MB * 64;  // 16-byte units of activations per stage
    constexpr int NT = NW * 64;
    constexpr int UPT = (STAGE_UNITS + NT - 1) / NT;  // the last round of a stage may be partial
    constexpr int WREGS = KK;                  // 16-byte weight loads per lane per stage

    __shared__ u32x4 lds[NBUF][STAGE_UNITS];  // ring of staged activation tiles (prefetch distance NBUF-1)

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, half = lane >> 5;
    const int nb = blockIdx.x * NW + wave;
    const bool active = nb < a.N / 32;
    const int split = blockIdx.y;
    const int mb_off = blockIdx.z * MR;  // first row block of this workgroup
    const int s0 = split * a.stages_per_split;
    const int s1 = min(a.n_stages, s0 + a.stages_per_split);
    const int kch = a.K / 128;

    // waves past the last column block work on block 0 and drop their result (keeps the loop branch-free)
    const u32x4* Wl = a.W + ((size_t)(active ? nb : 0) * kch) * 8 * 64 + lane;

    f32x16 acc[MR];
#pragma unroll
    for (int m = 0; m < MR; ++m)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[m][r] = 0.f;

    u32x4 w0[WREGS], w1[WREGS], w2[NBUF == 3 ? WREGS : 1], areg[UPT];

    auto load_w = [&](u32x4(&w)[WREGS], int st) {
#pragma unroll
        for (int j = 0; j < WREGS; ++j) w[j] = load_w16<STREAM>(Wl + ((size_t)st * WREGS + j) * 64);
    };
    auto load_a = [&](int st) {
#pragma unroll
        for (int i = 0; i < UPT; ++i) {
            const int u = min(i * NT + tid, STAGE_UNITS - 1);  // past the stage: re-read its last unit, never stored
            const int kk = u / (MB * 64), rem = u % (MB * 64);
            const int m = rem >> 6;  // operand block: hi plane of row block m, or lo plane of row block m - MR
            const int gb = m < MR ? mb_off + m : a.mb_rows + mb_off + (m - MR);
            areg[i] = a.A[((size_t)(st * KK + kk) * (2 * a.mb_rows) + gb) * 64 + (rem & 63)];
        }
    };
    auto store_a = [&](int buf) {
#pragma unroll
        for (int i = 0; i < UPT; ++i)
            if (STAGE_UNITS % NT == 0 || i * NT + tid < STAGE_UNITS) lds[buf][i * NT + tid] = areg[i];
    };
    auto compute = [&](int buf, const u32x4(&w)[WREGS]) {
        // A operands are read from LDS one k-step ahead of the MFMAs that use them; the 128-row
        // kernel reads them just in time instead: with the second fragment set it would not fit two
        // waves per SIMD, and the second wave hides more latency than the early read
        constexpr int AF = MB == 8 ? 1 : 2;
        u32x4 afr[AF][MB];
        if constexpr (AF == 2) {
#pragma unroll
            for (int m = 0; m < MB; ++m) afr[0][m] = lds[buf][m * 64 + lane];
        }
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            if constexpr (AF == 2) {
                if (kk + 1 < KK) {
#pragma unroll
                    for (int m = 0; m < MB; ++m) afr[(kk + 1) & 1][m] = lds[buf][((kk + 1) * MB + m) * 64 + lane];
                }
            } else {
#pragma unroll
                for (int m = 0; m < MB; ++m) afr[0][m] = lds[buf][(kk * MB + m) * 64 + lane];
            }
            __builtin_amdgcn_sched_barrier(0);
            const bf16x8 bfrag = __builtin_bit_cast(bf16x8, w[kk]);
#pragma unroll
            for (int pl = 0; pl < 2; ++pl)  // hi plane, then lo plane, into the same accumulators
#pragma unroll
                for (int m = 0; m < MR; ++m) {
                    const bf16x8 afrag = __builtin_bit_cast(bf16x8, afr[kk & (AF - 1)][pl * MR + m]);
                    acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afrag, bfrag, acc[m], 0, 0, 0);
                }
        }
    };

    // Steady state without branches around the loads, so that the requests of the following
    // stages stay in flight while this stage is computed; past the end the last stage is
    // re-read and never used.
    if (s0 < s1) {
        if constexpr (NBUF == 3) {
            auto phase = [&](const u32x4(&wc)[WREGS], u32x4(&wn)[WREGS], int bufc, int bufn, int st) {
                const int nx = min(st + 2, s1 - 1);
                load_a(nx);  // before the weights: the LDS store below then waits for these only
                load_w(wn, nx);
                compute(bufc, wc);
                store_a(bufn);
                __syncthreads();
            };
            const int sA = min(s0 + 1, s1 - 1);
            load_w(w0, s0);
            load_a(s0);
            store_a(0);
            load_w(w1, sA);
            load_a(sA);
            store_a(1);
            __syncthreads();
            for (int st = s0; st < s1; st += 3) {
                phase(w0, w2, 0, 2, st);
                if (st + 1 >= s1) break;
                phase(w1, w0, 1, 0, st + 1);
                if (st + 2 >= s1) break;
                phase(w2, w1, 2, 1, st + 2);
            }
        } else {
            load_w(w0, s0);
            load_a(s0);
            store_a(0);
            __syncthreads();
            for (int st = s0; st < s1; st += 2) {
                const int n1 = min(st + 1, s1 - 1);
                load_a(n1);
                load_w(w1, n1);
                compute(0, w0);
                store_a(1);
                __syncthreads();
                if (st + 1 >= s1) break;
                const int n2 = min(st + 2, s1 - 1);
                load_a(n2);
                load_w(w0, n2);
                compute(1, w1);
                store_a(0);
                __syncthreads();
            }
        }
    }
    if (!active) return;

    const int col = lane & 31;
    if constexpr (EPI == EPI_SWIGLU) {
        // The results leave as the tile the down projection reads: hi and lo plane, 16-byte units
        // of 8 consecutive u columns of one row, gathered through the wave's own piece of the (now idle)
        // activation ring.  Every wave has passed the barrier that follows the last stage.
        uint16_t* sw = reinterpret_cast<uint16_t*>(&lds[0][0]) + (size_t)wave * (MR * 32 * 16 * 2);
#pragma unroll
        for (int m = 0; m < MR; ++m) swiglu_strip<MR * 32>(acc[m], sw, m * 32);
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the wave's LDS writes have landed (no other wave reads them)
        __builtin_amdgcn_wave_barrier();
        u32x4* tile = reinterpret_cast<u32x4*>(a.out);
#pragma unroll
        for (int i = 0; i < MR * 2; ++i) {       // MR*32 rows x 2 units x 2 planes = MR*128 units, 64 lanes
            const int idx = i * 64 + lane;
            const int plane = idx / (MR * 64), rem = idx % (MR * 64), rl = rem >> 1, un = rem & 1;
            const int b = mb_off * 32 + rl;
            const u32x4 v = *reinterpret_cast<const u32x4*>(sw + ((size_t)plane * MR * 32 + rl) * 16 + un * 8);
            if (b < a.rows) tile[atile_unit(ATile{a.mb_rows}, plane, b, nb * 2 + un)] = v;
        }
    } else {
        float* o = a.out + (size_t)split * a.ld_rows * a.ldo + nb * 32 + col;
#pragma unroll
        for (int m = 0; m < MR; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int b = (mb_off + m) * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                if (b < a.rows) o[(size_t)b * a.ldo] = acc[m][r];
            }
    }
}

// ---------------------------------------------------------------------------------
// bf16 weights, more than 128 rows
// ---------------------------------------------------------------------------------
// Above 64 rows the projection is no longer bound by the weight stream, and the workgroup shape above would
// be bound by LDS just as much: there every operand fragment read from LDS feeds one matrix
// instruction (1 KiB per 32 cycles and SIMD = the 128 bytes per cycle the LDS delivers).  Here a
// wave owns 64 columns (two strips), so a fragment of the activations feeds two instructions.
// A workgroup is eight waves, two per SIMD, and covers 256 columns and 64 * MRW rows: wave (c, h)
// owns column pair c and row group h (MRW row blocks of 32; 2 in every launch: 128-row
// workgroups).  The two row groups of a column pair request the same weights (HBM sees them once).
// The activation stage is 64 wide (four k-steps) and shared by all waves.
// The next stage's weights are requested between the matrix instructions (all of them in front: gate/up at 256 rows 126 ->
// 120 us, the others 40.3 -> 38.7 on average).  Used above 128 rows.  Up to 128 rows the strip kernel stays (measured on the 14B shape at batch
// 128: gate/up 103 against 119 us, the rest equal).  A variant with four waves of 128 rows x 64
// columns, one per SIMD with its accumulators in the upper half of the register file, requests no
// weight twice but was 10 to 90 % slower: one wave per SIMD cannot cover its own waits.
template <int MRW, int EPI>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void proj_tall_kernel(ProjArgs a) {
    constexpr int RH = 2, NWC = 4;             // row groups and column pairs of a workgroup
    constexpr int MRT = RH * MRW;              // row blocks of the workgroup
    constexpr int MB = 2 * MRT;                // operand blocks of a k-step in LDS: hi planes, then lo planes
    constexpr int KK = 4;                      // k-steps per stage (64 of k)
    constexpr int STAGE_UNITS = KK * MB * 64;
    constexpr int NT = RH * NWC * 64;
    constexpr int NBUF = 2;                    // a third weight stage in registers does not fit beside 64 + 64 accumulators
    constexpr int UPT = (STAGE_UNITS + NT - 1) / NT;
    static_assert(STAGE_UNITS % NT == 0, "every thread stages the same number of units");
    __shared__ u32x4 lds_all[NBUF * STAGE_UNITS];

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, half = lane >> 5;
    const int wc = wave % NWC, rh = wave / NWC;
    const int cp = blockIdx.x * NWC + wc;      // column pair: strips 2 cp and 2 cp + 1
    const int n_strips = a.N / 32;
    const bool act0 = 2 * cp < n_strips, act1 = 2 * cp + 1 < n_strips;
    const int split = blockIdx.y;
    const int mb_off = blockIdx.z * MRT;       // first row block of this workgroup
    const int s0 = split * a.stages_per_split;
    const int s1 = min(a.n_stages, s0 + a.stages_per_split);
    const int kch = a.K / 128;

    // a stage is half a 128-wide chunk of the packed weights: four of its eight k-steps
    const u32x4* Wl0 = a.W + ((size_t)(act0 ? 2 * cp : 0) * kch) * 8 * 64 + lane;
    const u32x4* Wl1 = a.W + ((size_t)(act1 ? 2 * cp + 1 : 0) * kch) * 8 * 64 + lane;

    f32x16 acc[2][MRW];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int m = 0; m < MRW; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[s][m][r] = 0.f;

    u32x4 w0[2][KK], w1[2][KK], areg[UPT];

    auto load_w = [&](u32x4(&w)[2][KK], int st) {
        const size_t off = ((size_t)st * KK) * 64;   // in k-steps of 64 lanes
#pragma unroll
        for (int j = 0; j < KK; ++j) {
            w[0][j] = Wl0[off + (size_t)j * 64];
            w[1][j] = Wl1[off + (size_t)j * 64];
        }
    };
    auto load_a = [&](int st) {
#pragma unroll
        for (int i = 0; i < UPT; ++i) {
            const int u = i * NT + tid;
            const int kk = u / (MB * 64), rem = u % (MB * 64);
            const int m = rem >> 6;  // operand block: hi plane of row block m, or lo plane of row block m - MRT
            const int gb = m < MRT ? mb_off + m : a.mb_rows + mb_off + (m - MRT);
            areg[i] = a.A[((size_t)(st * KK + kk) * (2 * a.mb_rows) + gb) * 64 + (rem & 63)];
        }
    };
    auto store_a = [&](int buf) {
#pragma unroll
        for (int i = 0; i < UPT; ++i) lds_all[buf * STAGE_UNITS + i * NT + tid] = areg[i];
    };
    // the next stage's weights are requested between the k-steps' matrix instructions
    auto compute = [&](int buf, const u32x4(&w)[2][KK], u32x4(&wn)[2][KK], int nst) {
        // this wave's operand blocks of a k-step: hi and lo plane of its MRW row blocks
        const u32x4* src = lds_all + buf * STAGE_UNITS + lane;
        u32x4 afr[2][2 * MRW];
        auto read_a = [&](int kk, u32x4(&dst)[2 * MRW]) {
#pragma unroll
            for (int pl = 0; pl < 2; ++pl)
#pragma unroll
                for (int m = 0; m < MRW; ++m) dst[pl * MRW + m] = src[(kk * MB + pl * MRT + rh * MRW + m) * 64];
        };
        read_a(0, afr[0]);
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            if (kk + 1 < KK) read_a(kk + 1, afr[(kk + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const bf16x8 bfrag = __builtin_bit_cast(bf16x8, w[s][kk]);
#pragma unroll
                for (int pl = 0; pl < 2; ++pl)  // hi plane, then lo plane, into the same accumulators
#pragma unroll
                    for (int m = 0; m < MRW; ++m) {
                        const bf16x8 afrag = __builtin_bit_cast(bf16x8, afr[kk & 1][pl * MRW + m]);
                        acc[s][m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afrag, bfrag, acc[s][m], 0, 0, 0);
                    }
                __builtin_amdgcn_sched_barrier(0);
                const size_t off = ((size_t)nst * KK + kk) * 64;
                wn[s][kk] = s ? Wl1[off] : Wl0[off];
            }
        }
    };

    if (s0 < s1) {
        load_w(w0, s0);
        load_a(s0);
        store_a(0);
        __syncthreads();
        for (int st = s0; st < s1; st += 2) {
            const int n1 = min(st + 1, s1 - 1);
            load_a(n1);
            compute(0, w0, w1, n1);
            store_a(1);
            __syncthreads();
            if (st + 1 >= s1) break;
            const int n2 = min(st + 2, s1 - 1);
            load_a(n2);
            compute(1, w1, w0, n2);
            store_a(0);
            __syncthreads();
        }
    }

    const int col = lane & 31;
    if constexpr (EPI == EPI_SWIGLU) {
        // The results leave as the tile the down projection reads: hi and lo plane, 16-byte units
        // of 8 consecutive u columns of one row, gathered through the wave's own piece of the (now idle)
        // activation ring.  Every wave has passed the barrier that follows the last stage.
        uint16_t* sw = reinterpret_cast<uint16_t*>(lds_all) + (size_t)wave * (MRW * 32 * 16 * 2);
        u32x4* tile = reinterpret_cast<u32x4*>(a.out);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int nb = 2 * cp + s;
#pragma unroll
            for (int m = 0; m < MRW; ++m) swiglu_strip<MRW * 32>(acc[s][m], sw, m * 32);
            __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the wave's LDS writes have landed (no other wave reads them)
            __builtin_amdgcn_wave_barrier();
            if (nb < n_strips) {
#pragma unroll
                for (int i = 0; i < MRW * 2; ++i) {       // MRW*32 rows x 2 units x 2 planes = MRW*128 units, 64 lanes
                    const int idx = i * 64 + lane;
                    const int plane = idx / (MRW * 64), rem = idx % (MRW * 64), rl = rem >> 1, un = rem & 1;
                    const int b = (mb_off + rh * MRW) * 32 + rl;
                    const u32x4 v = *reinterpret_cast<const u32x4*>(sw + ((size_t)plane * MRW * 32 + rl) * 16 + un * 8);
                    if (b < a.rows) tile[atile_unit(ATile{a.mb_rows}, plane, b, nb * 2 + un)] = v;
                }
            }
            __builtin_amdgcn_s_waitcnt(0xc07f);  // the reads are done before the second strip overwrites the piece
            __builtin_amdgcn_wave_barrier();
        }
    } else {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int nb = 2 * cp + s;
            if (nb >= n_strips) continue;
            float* o = a.out + (size_t)split * a.ld_rows * a.ldo + nb * 32 + col;
#pragma unroll
            for (int m = 0; m < MRW; ++m)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int b = (mb_off + rh * MRW + m) * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                    if (b < a.rows) o[(size_t)b * a.ldo] = acc[s][m][r];
                }
        }
    }
}

// ---------------------------------------------------------------------------------
// bf16 weights, many rows (prefill blocks; the vocabulary projection above 128 rows)
// ---------------------------------------------------------------------------------
// Bound by the matrix cores (and the clock they leave: see the figures).  A workgroup of eight waves covers 256 rows x
// 256 columns; a wave owns 64 rows x 128 columns, so that the eight fragments it reads from LDS per k-step feed sixteen
// matrix instructions (both activation planes against the same weight fragment).  Both operands are stored in
// fragment order, so a stage (two k-steps, 48 fragments of 1 KiB) goes from memory straight into one of three LDS
// slots, two stages ahead, without passing through registers.  The requests leave between the matrix instructions,
// where the memory pipeline's back pressure is covered: all of a stage's requests at its start cost 10 %.
// Larger tiles than the kernel above because what limits there is the traffic from L2 into the compute units:
// 24 bytes per cycle here against 47.  Measured, 28 672 x 4096, both planes counted: 1024 rows 384 us on average in a prefill (368
// the shortest) = 1.25 PFLOP/s, 2048 rows 729 (713) = 1.32 (four / eight launches of the 128 x 256 kernel: 505 / 1010 us; the
// instructions alone, no loads: 322 / 591; the same code on zeros, which draw less power and leave the clock up: 294 / 583).
// CB: 32-column strips of a workgroup, eight or, where that makes whole rounds, fewer (wide_pick_strips).  RAGGED: row blocks without a row are
// left out of the products (launch_proj_wide).
// Measured and left out: 128 x 256 tiles in this scheme (1024 rows 430 us; at 256 rows no faster than the kernel
// above), four or five slots, a deeper ring for the weights than for the activations, streaming loads for the
// weights (the row tiles share them through L2: 775 us), a rotated start along k, other workgroup orders.
template <int EPI, int CB, bool RAGGED>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void proj_wide_kernel(ProjArgs a) {
    constexpr int RB = 8, CS = 8;                       // row blocks of a workgroup, and places for its column strips in a slot
    constexpr int S0 = (CB + 1) / 2;                    // strips of the waves of column half 0; the others have CB - S0
    constexpr int AF = 2 * 2 * RB, WF = 2 * CS;         // operand fragments (1 KiB) of a stage: two k-steps
    constexpr int STAGE_UNITS = (AF + WF) * 64;         // 16-byte units (48 KiB)
    constexpr int NBUF = 3;
    constexpr int WA = AF / 8, PER = WA + WF / 8;       // fragments a wave fetches per stage: four of A, two of W
    __shared__ u32x4 lds_all[NBUF * STAGE_UNITS];

    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // column half, 64-row group; the two waves of a SIMD (w and w + 4) are of different halves, which may differ by a strip
    const int ch = (wave ^ (wave >> 2)) & 1, rh = wave >> 1;
    const bool short_half = CB % 2 && ch == 1;
    // row blocks of this wave that hold a row (none: 0 or less)
    const int blocks = RAGGED ? min(2, (a.rows - ((int)blockIdx.z * RB + rh * 2) * 32 + 31) / 32) : 2;
    const int n_strips = a.N / 32;
    const int strip0 = blockIdx.x * CB;
    const int split = blockIdx.y;
    const int mb_off = blockIdx.z * RB;
    const int s0 = split * a.stages_per_split;
    const int s1 = min(a.n_stages, s0 + a.stages_per_split);
    const int n = s1 - s0;
    const size_t kch8 = (size_t)(a.K / 128) * 8;        // k-steps of a strip

    // what this wave fetches of every stage, activations first
    const u32x4* src[PER];
    uint32_t dst[PER];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) u32x4*)lds_all;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (i < WA) {
            const int f = wave * WA + i, ks = f / (2 * RB), blk = f % (2 * RB);
            const int gb = blk < RB ? mb_off + blk : a.mb_rows + mb_off + (blk - RB);  // hi planes, then lo planes
            src[i] = a.A + ((size_t)(s0 * 2 + ks) * (2 * a.mb_rows) + gb) * 64;
            dst[i] = lds0 + f * 1024;
        } else {
            const int f = min(wave * (WF / 8) + (i - WA), 2 * CB - 1), ks = f / CB, blk = f % CB;   // past the last: that one again, the same bytes
            const int strip = min(strip0 + blk, n_strips - 1);  // past the last strip: any valid one, its result is dropped
            src[i] = a.W + ((size_t)strip * kch8 + s0 * 2 + ks) * 64;
            dst[i] = lds0 + (AF + ks * CS + blk) * 1024;
        }
    }
    const size_t step_a = (size_t)4 * a.mb_rows * 64, step_w = 128;  // units from one stage to the next
    uint32_t fill = 0;                                  // ring offset and number of the stage that is requested next
    int fill_st = 0;
    auto issue = [&](int i) {                           // past the end the last stage again (it is not read)
        lds_dma16(src[i], lane * 16, dst[i] + fill);
        if (fill_st + 1 < n) src[i] += i < WA ? step_a : step_w;
    };
    auto issued = [&]() {
        fill += STAGE_UNITS * 16;
        if (fill == NBUF * STAGE_UNITS * 16) fill = 0;
        ++fill_st;
    };
    f32x16 acc[S0][2];
#pragma unroll
    for (int s = 0; s < S0; ++s)
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[s][m][r] = 0.f;

    struct Frags {
        u32x4 a[2][2], w[S0];
    };
    int at = 0;                                         // ring slot that is read
    auto read = [&](Frags& f, int ks) {
        const u32x4* p = lds_all + at * STAGE_UNITS + lane;
#pragma unroll
        for (int pl = 0; pl < 2; ++pl)
#pragma unroll
            for (int m = 0; m < 2; ++m) f.a[pl][m] = p[(ks * 2 * RB + pl * RB + rh * 2 + m) * 64];
#pragma unroll
        for (int s = 0; s < S0; ++s) f.w[s] = p[(AF + ks * CS + ch * S0 + s) * 64];   // past a short half's strips: not used
    };
    // 4 S0 matrix instructions (16 for 256 columns), the requests i0 .. i0 + 2 of the stage being fetched between them
    auto mma = [&](const Frags& f, int i0) {
#pragma unroll
        for (int pl = 0; pl < 2; ++pl)
#pragma unroll
            for (int s = 0; s < S0; ++s) {
                if ((s + 1 < S0 || !short_half) && (!RAGGED || blocks > 0)) {
#pragma unroll
                    for (int m = 0; m < 2; ++m)
                        if (!RAGGED || m < blocks)
                            acc[s][m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f.a[pl][m]),
                                                                          __builtin_bit_cast(bf16x8, f.w[s]), acc[s][m], 0, 0, 0);
                }
                const int g = pl * S0 + s;
                if ((g & 1) && g < 6) {
                    __builtin_amdgcn_sched_barrier(0);
                    issue(i0 + (g >> 1));
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
    };
    // The oldest stage in flight has landed for every wave, and every wave has its fragments of the stage before in
    // registers, so that stage's slot may be overwritten.
    auto enter = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0xc07f);             // lgkmcnt(0)
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(PER * (NBUF - 2)) : "memory");
    };
    if (n > 0) {
#pragma unroll
        for (int b = 0; b < NBUF - 1; ++b) {
#pragma unroll
            for (int i = 0; i < PER; ++i) issue(i);
            issued();
        }
        Frags f0, f1;
        enter();
        read(f0, 0);
        for (int st = 0; st < n; ++st) {
            read(f1, 1);
            __builtin_amdgcn_sched_barrier(0);
            mma(f0, 0);
            mma(f1, 3);
            issued();
            at = at + 1 == NBUF ? 0 : at + 1;
            if (st + 1 < n) {
                enter();
                read(f0, 0);
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");  // nothing is in flight into LDS any more
    const int my_strip = strip0 + ch * S0, my_end = min(n_strips, strip0 + (ch ? CB : S0));
    const int col = lane & 31, row0 = (mb_off + rh * 2) * 32;
    if constexpr (EPI == EPI_SWIGLU) {
        // The results leave as the tile the down projection reads: hi and lo plane, 16-byte units
        // of 8 consecutive u columns of one row, gathered through the wave's own piece of the idle ring.
        uint16_t* sw = reinterpret_cast<uint16_t*>(lds_all) + (size_t)wave * (2 * 64 * 16);
        u32x4* tile = reinterpret_cast<u32x4*>(a.out);
#pragma unroll
        for (int s = 0; s < S0; ++s) {
            const int nb = my_strip + s;
#pragma unroll
            for (int m = 0; m < 2; ++m) swiglu_strip<64>(acc[s][m], sw, m * 32);
            __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the wave's LDS writes have landed (no other wave reads them)
            __builtin_amdgcn_wave_barrier();
            if (nb < my_end) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {    // 64 rows x 2 units x 2 planes = 256 units, 64 lanes
                    const int idx = i * 64 + lane;
                    const int plane = idx >> 7, rem = idx & 127, rl = rem >> 1, un = rem & 1;
                    const u32x4 v = *reinterpret_cast<const u32x4*>(sw + ((size_t)plane * 64 + rl) * 16 + un * 8);
                    if (row0 + rl < a.rows) tile[atile_unit(ATile{a.mb_rows}, plane, row0 + rl, nb * 2 + un)] = v;
                }
            }
            __builtin_amdgcn_s_waitcnt(0xc07f);  // the reads are done before the next strip overwrites the piece
            __builtin_amdgcn_wave_barrier();
        }
    } else {
#pragma unroll
        for (int s = 0; s < S0; ++s) {
            const int nb = my_strip + s;
            if (nb >= my_end) continue;
            float* o = a.out + (size_t)split * a.ld_rows * a.ldo + nb * 32 + col;
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int b = row0 + m * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                    if (b < a.rows) o[(size_t)b * a.ldo] = acc[s][m][r];
                }
        }
    }
}

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

// 4-bit weights: a 32-row tile per workgroup (see proj_tiling), one stage = one 128-wide group = four int8 MFMA k-steps.
// Bound by what a short launch has around its steady state (latency of the stages, the vector epilogue), so stages are
// requested far ahead without registers to hold them: the activations and their scales go straight into one of three LDS
// slots, two stages ahead, and the registers that this frees hold the codes three stages ahead instead of two.  8B shape,
// against both through registers two stages ahead (us): 5 rows qkv 7.3 -> 6.8, gate/up 17.2 -> 16.1, o and down 10.3 ->
// 8.5 on average; 64 rows gate/up 30.2 -> 29.2; bit-identical.  Codes four and activations three stages ahead (128
// registers): 64 rows 28.7, 5 rows 17.0, not better.
// OCT: row octets of a tile that the epilogue scales: 4, or as many as a launch of at most 16 rows has rows in (the epilogue
// is most of the vector instructions: gate/up at 5 rows 19.1 -> 17.2 us, the step of 8 layers 924 -> 885).
template <int NW, int OCT>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2, 4)))
void proj_w4_kernel(ProjArgs a) {
    constexpr int STEPS = 4, PA = 2, PW = 3, NBUF = PA + 1;
    constexpr int FR = STEPS * 2, ITEMS = FR + 1, PER = (ITEMS + NW - 1) / NW;  // 1 KiB fragments of a stage, and its scales
    constexpr int STAGE_BYTES = FR * 1024 + 256;
    __shared__ __attribute__((aligned(16))) uint8_t lds[NBUF * STAGE_BYTES];

    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nb = blockIdx.x * NW + wave;
    const bool active = nb < a.N / 32;
    const int split = blockIdx.y;
    const int mb = blockIdx.z;
    const int s0 = split * a.stages_per_split;
    const int n = min(a.n_stages, s0 + a.stages_per_split) - s0;
    const int kch = a.K / 128;

    // waves past the last column block work on block 0 and drop their result (keeps the loop branch-free)
    const u32x4* Wl = a.W + ((size_t)(active ? nb : 0) * kch + s0) * 2 * 64 + lane;
    const uint32_t* SZl = a.SZ + ((size_t)(active ? nb : 0) * (a.s_only ? (kch + 1) >> 1 : kch)) * 32 + (lane & 31);

    // what this wave fetches of every stage: fragments (k-step, plane), and as the last item the rows' (scale, sum) pairs
    const uint8_t* src[PER];
    uint32_t dst[PER], step[PER];
    bool frag[PER];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int f = min(wave * PER + i, ITEMS - 1);   // past the last: that one again, the same bytes
        frag[i] = f < FR;
        src[i] = frag[i] ? (const uint8_t*)(a.A + ((size_t)(s0 * FR + f) * a.mb_rows + mb) * 64)
                         : (const uint8_t*)(a.qscale + ((size_t)s0 * a.mb_rows + mb) * 64);
        step[i] = frag[i] ? FR * a.mb_rows * 1024 : a.mb_rows * 256;
        dst[i] = lds0 + f * 1024;
    }
    int fill = 0, fill_st = 0;
    auto fetch = [&]() {                                // the next stage; past the end the last one again (it is not read)
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (frag[i]) lds_dma16(src[i], lane * 16, dst[i] + fill);
            else lds_dma4(src[i], lane * 4, dst[i] + fill);
            if (fill_st + 1 < n) src[i] += step[i];
        }
        ++fill_st;
        fill = fill + STAGE_BYTES == NBUF * STAGE_BYTES ? 0 : fill + STAGE_BYTES;
    };
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    u32x4 w[PW + 1][2];
    uint32_t sz[PW + 1];
    auto load_w = [&](int slot, int st) {
        const int t = min(st, n - 1);
        w[slot][0] = Wl[(size_t)t * 2 * 64];
        w[slot][1] = Wl[((size_t)t * 2 + 1) * 64];
        sz[slot] = SZl[(size_t)(a.s_only ? (s0 + t) >> 1 : s0 + t) * 32];
    };
    int at = 0;
    auto compute = [&](int slot, int st) {
        const u32x4* A = reinterpret_cast<const u32x4*>(lds + at) + lane;
        i32x16 ih, il;
        u32x4 afr[2][2];  // operands of one k-step (both planes), read one step ahead
        afr[0][0] = A[0];
        afr[0][1] = A[64];
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            if (s + 1 < STEPS) {
                afr[(s + 1) & 1][0] = A[(s + 1) * 128];
                afr[(s + 1) & 1][1] = A[(s + 1) * 128 + 64];
            }
            __builtin_amdgcn_sched_barrier(0);
            const uint32_t wa = w[slot][s >> 1][(s & 1) * 2], wb = w[slot][s >> 1][(s & 1) * 2 + 1];
            const i32x4 bfrag = {(int)(wa & 0x0F0F0F0Fu), (int)((wa >> 4) & 0x0F0F0F0Fu), (int)(wb & 0x0F0F0F0Fu),
                                 (int)((wb >> 4) & 0x0F0F0F0Fu)};
            const i32x4 ah = __builtin_bit_cast(i32x4, afr[s & 1][0]), al = __builtin_bit_cast(i32x4, afr[s & 1][1]);
            if (s == 0) {
                i32x16 zero;
#pragma unroll
                for (int r = 0; r < 16; ++r) zero[r] = 0;
                ih = __builtin_amdgcn_mfma_i32_32x32x32_i8(ah, bfrag, zero, 0, 0, 0);
                il = __builtin_amdgcn_mfma_i32_32x32x32_i8(al, bfrag, zero, 0, 0, 0);
            } else {
                ih = __builtin_amdgcn_mfma_i32_32x32x32_i8(ah, bfrag, ih, 0, 0, 0);
                il = __builtin_amdgcn_mfma_i32_32x32x32_i8(al, bfrag, il, 0, 0, 0);
            }
        }
        // scale-only layout: pick this group's half of the dword; the zero point is 8 everywhere
        const uint32_t szg = a.s_only ? (((sz[slot] >> (16 * ((s0 + st) & 1))) & 0xffffu) | 0x48000000u) : sz[slot];
        const __half2 h2 = __builtin_bit_cast(__half2, szg);
        const float sc = __low2float(h2);
        const int nzi = -(int)__high2float(h2);  // zero points are integer codes (Appendix A.1)
        const u32x4* Q = reinterpret_cast<const u32x4*>(lds + at + FR * 1024) + 2 * half;
#pragma unroll
        for (int rr = 0; rr < OCT; ++rr) {
            const u32x4 q01 = Q[rr * 4], q23 = Q[rr * 4 + 1];   // (scale, sum of integers) of four rows
            const float sx[4] = {__uint_as_float(q01[0]), __uint_as_float(q01[2]), __uint_as_float(q23[0]), __uint_as_float(q23[2])};
            const int xs[4] = {(int)q01[1], (int)q01[3], (int)q23[1], (int)q23[3]};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int e = rr * 4 + q;
                int tot = (ih[e] << 8) + il[e];
                asm("v_mad_i32_i24 %0, %1, %2, %0" : "+v"(tot) : "v"(nzi), "v"(xs[q]));  // tot -= Z * sum xi, one instruction
                acc[e] = fmaf((float)tot, sc * sx[q], acc[e]);
            }
        }
        at = at + STAGE_BYTES == NBUF * STAGE_BYTES ? 0 : at + STAGE_BYTES;
    };
    if (n > 0) {
#pragma unroll
        for (int i = 0; i < PA; ++i) fetch();
#pragma unroll
        for (int i = 0; i < PW; ++i) load_w(i, i);
        auto phase = [&](int slot, int st) {
            // stage st of the activations has landed for every wave, and everybody is done with stage st - 1
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(0xc07f);
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(3 + (PA - 1) * (PER + 3)) : "memory");
            fetch();
            load_w((slot + PW) % (PW + 1), st + PW);
            __builtin_amdgcn_sched_barrier(0);
            compute(slot, st);
        };
        for (int st = 0; st < n;) {
#pragma unroll
            for (int i = 0; i <= PW; ++i) {
                phase(i, st);
                if (++st >= n) break;
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // nothing is in flight into LDS when the workgroup ends
    if (!active) return;
    const int col = lane & 31;
    float* o = a.out + (size_t)split * a.ld_rows * a.ldo + nb * 32 + col;
#pragma unroll
    for (int r = 0; r < OCT * 4; ++r) {
        const int b = mb * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
        if (b < a.rows) o[(size_t)b * a.ldo] = acc[r];
    }
}

static hipError_t launch_proj_w4(const ProjArgs& a, int nw, int splits, int mtiles, hipStream_t st) {
    const auto go = [&](auto nwc) {
        constexpr int NW = decltype(nwc)::value;
        dim3 grid((a.N / 32 + NW - 1) / NW, splits, mtiles), block(NW * 64);
        if (a.rows <= 8) hipLaunchKernelGGL((proj_w4_kernel<NW, 1>), grid, block, 0, st, a);
        else if (a.rows <= 16) hipLaunchKernelGGL((proj_w4_kernel<NW, 2>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((proj_w4_kernel<NW, 4>), grid, block, 0, st, a);
        return hipGetLastError();
    };
    switch (nw) {
    case 4: return go(std::integral_constant<int, 4>{});
    case 5: return go(std::integral_constant<int, 5>{});
    case 6: return go(std::integral_constant<int, 6>{});
    case 7: return go(std::integral_constant<int, 7>{});
    }
    return hipErrorInvalidValue;
}

template <int MB, int KS, int NW, bool STREAM>
static hipError_t launch_proj_t(const ProjArgs& a, int epilogue, int splits, int mtiles, hipStream_t st) {
    constexpr int NBUF = (MB * KS * 64 * 3 <= 49152) ? 3 : 2;  // LDS ring: 3 stages when they fit in 48 KB
    dim3 grid((a.N / 32 + NW - 1) / NW, splits, mtiles), block(NW * 64);
    if (epilogue == EPI_SWIGLU) {
        if (splits != 1) return hipErrorInvalidValue;
        hipLaunchKernelGGL((proj_kernel<MB, KS, NW, EPI_SWIGLU, NBUF, STREAM>), grid, block, 0, st, a);
        return hipGetLastError();
    }
    if (epilogue != EPI_STORE) return hipErrorInvalidValue;
    hipLaunchKernelGGL((proj_kernel<MB, KS, NW, EPI_STORE, NBUF, STREAM>), grid, block, 0, st, a);
    return hipGetLastError();
}

static hipError_t launch_proj_tall(const ProjArgs& a, int epilogue, int splits, int mtiles, hipStream_t st) {
    const int pairs = (a.N / 32 + 1) / 2;
    dim3 grid((pairs + 3) / 4, splits, mtiles);
    if (epilogue == EPI_SWIGLU) {
        if (splits != 1) return hipErrorInvalidValue;
        hipLaunchKernelGGL((proj_tall_kernel<2, EPI_SWIGLU>), grid, dim3(512), 0, st, a);
        return hipGetLastError();
    }
    if (epilogue != EPI_STORE) return hipErrorInvalidValue;
    hipLaunchKernelGGL((proj_tall_kernel<2, EPI_STORE>), grid, dim3(512), 0, st, a);
    return hipGetLastError();
}

static hipError_t launch_proj_wide(const ProjArgs& a, int epilogue, int cb, int splits, hipStream_t st) {
    const auto go = [&](auto cbc) {
        constexpr int CB = decltype(cbc)::value;
        dim3 grid((a.N / 32 + CB - 1) / CB, splits, (a.rows + 255) / 256);
        // Row blocks without a row cost no matrix instruction where they are an eighth of the launch or more; below that the branches
        // cost more (4 layers of the 8B shape, left out: 260 / 400 / 800 (14B) tokens with 44 / 19 / 22 % of them 1864 / 1905 / 4311 ->
        // 1677 / 1861 / 4154 us, 1100 / 1300 with 13 / 15 % 4181 / 5051 -> 4152 / 5014, 900 with 9 % 3419 -> 3435, 1200 (14B) with 5 %
        // 5503 -> 5594, 1500 with 2 % 5170 -> 5298; a 4-bit step of 150 requests,
        // whose vocabulary has three blocks of eight left out, 3288 -> 3228).  In the one row tile of a vocabulary a single block of
        // eight is not enough (200 rows, vocabulary 65 536 of hidden 4096 / 128 256 of hidden 1024: 200 / 114 -> 213 / 118 us).
        const int row_blocks = (a.rows + 31) / 32, launched = (a.rows + 255) / 256 * 8;
        const bool ragged = (launched - row_blocks) * (launched == 8 ? 4 : 8) >= launched;
        if (epilogue == EPI_SWIGLU) {
            if (splits != 1) return hipErrorInvalidValue;
            if (ragged) hipLaunchKernelGGL((proj_wide_kernel<EPI_SWIGLU, CB, true>), grid, dim3(512), 0, st, a);
            else hipLaunchKernelGGL((proj_wide_kernel<EPI_SWIGLU, CB, false>), grid, dim3(512), 0, st, a);
            return hipGetLastError();
        }
        if (epilogue != EPI_STORE) return hipErrorInvalidValue;
        if (ragged) hipLaunchKernelGGL((proj_wide_kernel<EPI_STORE, CB, true>), grid, dim3(512), 0, st, a);
        else hipLaunchKernelGGL((proj_wide_kernel<EPI_STORE, CB, false>), grid, dim3(512), 0, st, a);
        return hipGetLastError();
    };
    switch (cb) {
    case 5: return go(std::integral_constant<int, 5>{});
    case 6: return go(std::integral_constant<int, 6>{});
    case 7: return go(std::integral_constant<int, 7>{});
    case 8: return go(std::integral_constant<int, 8>{});
    }
    return hipErrorInvalidValue;
}

// Split-K factor of the launch above 128 rows (bf16; workgroups of 128 rows x 256 columns).  All workgroups do
// equal work and one round of at most 256 of them is wanted: the largest split that stays within the round
// (each split costs a slab of partial sums, but the matrix-core time of a workgroup goes with its stages;
// measured on the 8B shape at 256 rows: qkv 5 splits 32.7 us against 37.7 with 4, down 8 against 4: 64 / 125).
static int tall_pick_splits(const Mat& W, int rows, int max_splits) {
    const int pairs = (W.N / 32 + 1) / 2, stages = W.K / 64, colwgs = (pairs + 3) / 4;
    const int mtiles = (atile_for_rows(rows).MB + 3) / 4;
    int best = 1;
    for (int s = 1; s <= max(1, min(max_splits, stages / 4)); ++s) {
        const int sps = (stages + s - 1) / s;
        if ((stages + sps - 1) / sps != s) continue;
        if ((long long)colwgs * mtiles * s <= 256) best = s;
    }
    return best;
}

static constexpr int chunks_per_split(int kch, int splits) { return (kch + splits - 1) / splits; }

// Waves per workgroup (each wave owns 32 columns) and split-K factor.  A compute unit's share of
// the HBM bandwidth does not grow with the number of workgroups it hosts, so the launch is only
// as fast as the most loaded unit: the pair is chosen to spread the weight bytes evenly over the
// 256 compute units (N = 6144 -> 6 waves x 8 splits, N = 4096 -> 4 x 8, ...), with a
// fixed charge per workgroup for filling and draining its pipeline.  Depends on the matrix and the
// row-count class only.  The bf16 kernel above 64 rows keeps 4 waves; 4-bit launches of several row tiles have
// a rule of their own (w4_tiles_pick).
struct ProjShape {
    int nw, splits;
};
// Row tiling: operand blocks per workgroup (2 planes x 32-row blocks) and row tiles per launch.
// bf16 weights: up to 64 rows one tile holds all rows; above, 128-row tiles (every tile streams the
// weights from HBM again).  4-bit weights: 32-row tiles at every batch size.  Their kernel is bound by
// its vector-ALU epilogue and by the wait for the matrix cores between epilogues, not by the weight
// stream (a quarter of the bytes, and the row tiles of a column strip run side by side and share
// their fetches); with one row block a wave needs 128 registers instead of 230, four waves share a
// SIMD instead of two and cover each other's waits.  Only tiles that hold a row are launched (150 rows: 5 of the
// activation tiling's 8, gate/up 102 -> 81 us) (8B shape, qkv / o / gate-up / down in us: batch 64
// 16.2 / 11.9 / 32.7 / 21.6 -> 15.0 / 11.1 / 30.0 / 20.5; batch 256 30.9 / 22.7 / 104.6 / 60.2 -> 27.8 / 20.6 /
// 90.9 / 50.7; results bit-identical).
struct ProjTiling {
    int mb, mtiles;
};
static ProjTiling proj_tiling(const Mat& W, int rows) {
    const int mbr = atile_for_rows(rows).MB;  // 32-row blocks of the activation tiling: 1, 2, 4 or a multiple of 8
    if (W.kind == MAT_W4_PACKED) return ProjTiling{2, (rows + 31) / 32};  // no tile without a row
    if (mbr <= 2) return ProjTiling{2 * mbr, 1};
    return ProjTiling{8, mbr / 4};
}
// Beside its strips a workgroup costs what it takes to start and end (six strip stages).
static constexpr long long proj_cost(int strips, int kch, int mtiles, int nw, int s, int ends = 6) {
    const int cps = chunks_per_split(kch, s), real_s = (kch + cps - 1) / cps;
    const long long wgs = (long long)((strips + nw - 1) / nw) * real_s * mtiles;
    const long long rounds = (wgs + 255) / 256;
    return rounds * ((long long)nw * cps + ends) * 16 + real_s;  // ties: fewer splits
}
// 4-bit weights with more than one 32-row tile: several workgroups share a compute unit (16 waves at 128
// registers), so the launch wants two to four times 256 workgroups rather than exactly 256.  Four waves per
// workgroup (seven for a matrix of 512 strips or more while there are only two row tiles), and the smallest
// split into equal shares that gives at least 512 workgroups without leaving a workgroup more than 32 stages.  Measured on the 8B
// shape (us, best of the shapes tried): batch 64 qkv 4 x 8: 13.5 (6 x 8: 14.7, 4 x 4: 15.3), o 4 x 8: 10.8
// (4 x 4: 12.0, 4 x 16: 12.6), gate/up 7 x 2: 30.0 (4 x 2: 31.8, 7 x 1: 35.6), down 4 x 8: 19.7 (4 x 4: 26.8);
// batch 256 qkv 4 x 2: 25.8 (4 x 4: 27.5, 4 x 8: 30.3), o 4 x 4: 20.4, gate/up 4 x 1: 92.4 (4 x 2: 95.4, 4 x 4: 105),
// down 4 x 4: 49.4 (4 x 2: 52.4, 4 x 8: 51.3).
static ProjShape w4_tiles_pick(const Mat& W, int mtiles, int max_splits) {
    const int strips = W.N / 32, kch = W.K / 128;
    const int nw = (strips >= 512 && mtiles <= 2) ? 7 : 4;
    const long long colwgs = (strips + nw - 1) / nw;
    ProjShape best{nw, 1};
    for (int s = 1; s <= max(1, min(max_splits, kch / 2)); ++s) {
        if (kch % s) continue;  // equal shares only: the launch ends with its longest workgroup
        best = ProjShape{nw, s};
        if (colwgs * mtiles * s >= 448 && kch / s <= 32) break;  // "at least 512", with a little give
    }
    return best;
}
static ProjShape proj_pick(const Mat& W, int rows, int max_splits) {
    const int strips = W.N / 32, kch = W.K / 128;
    const ProjTiling t = proj_tiling(W, rows);
    const int mtiles = t.mtiles;
    // by the activation tiling's row blocks rather than the tiles that are launched: a row's sums then depend on the class of the
    // row count alone (65 to 128, 129 to 256), not on the rows beside it (8B shape, by launched tiles instead: 66 / 150 / 224 rows
    // 1412 / 2064 / 2546 us a step against 1432 / 2078 / 2546)
    if (W.kind == MAT_W4_PACKED && mtiles >= 2) return w4_tiles_pick(W, atile_for_rows(rows).MB, max_splits);
    const int smax = max(1, min(max_splits, kch / 2));
    ProjShape best{4, 1};
    long long best_cost = -1;
    for (int nw = 4; nw <= (t.mb <= 4 ? 7 : 4); ++nw)
        for (int s = 1; s <= smax; ++s) {
            const long long c = proj_cost(strips, kch, mtiles, nw, s);
            if (best_cost < 0 || c < best_cost) {
                best_cost = c;
                const int cps = chunks_per_split(kch, s);
                best = ProjShape{nw, (kch + cps - 1) / cps};
            }
        }
    return best;
}

// Which kernel multiplies more than 128 rows (bf16).  256 x 256 tiles want whole rounds of 256 workgroups without a
// split along k: a prefill block (rows > 256) and a vocabulary projection have them.  A batch's other projections do not: the
// 128 x 256 tiles of the tall kernel (8B shape, 256 rows: o, q/k/v, down, gate/up 24 / 32 / 60 / 115 us) beat the wide kernel,
// split finer, by 27 to 40 %.
// Columns that just exceed one round pay a second one, and more so the shorter k is: there the strip kernel stays (128-row tiles,
// two workgroups on a compute unit).  Strip -> wide kernel at 256 rows (us): hidden 1024 with 66 048 / 80 000 / 84 000 / 98 304
// columns 92 -> 98 / 96 -> 99 / 106 -> 100 / 120 -> 109, hidden 2048 with 66 048 / 72 032 /
// 76 000 / 98 304 175 -> 185 / 186 -> 186 / 190 -> 187 / 242 -> 201, hidden 4096 with 65 568 / 80 000 / 128 256 359 -> 350 / 403 ->
// 374 / 635 -> 458, one whole round (65 536) against the tall kernel 311 -> 233; each with the
// tiling of its input (the last 458 are 400 in a step).
static bool use_wide(const Mat& W, int rows) {
    if (W.kind != MAT_BF16_PACKED) return false;
    const int tiles = (W.N / 32 + 7) / 8;
    return rows > kMaxBatchTile || (rows > 128 && (tiles == 256 || (tiles > 256 && (W.K >= 4096 || tiles >= (W.K >= 2048 ? 288 : 320)))));
}
static bool use_tall(const Mat& W, int rows) {
    return W.kind == MAT_BF16_PACKED && rows > 128 && !use_wide(W, rows) && (W.N / 32 + 7) / 8 <= 256;
}

// Split-K factor of a wide launch: whole rounds of 256 workgroups of eight strips cost stages x 0.95 us (2048 cycles of matrix
// instructions) plus about 8 us each, a split the writing and reading of its slab.  The factor sets the order of the sums, so
// it does not follow the tile width below: chosen together with it, o at 1024 rows went from four slabs to two and with its norm from 91 to
// 102 us, down at 768 / 1536 rows from 163 / 319 to 186 / 342 (8B shape), at 1024 rows from 251 to 268 (14B shape).
static int wide_pick_splits(const Mat& W, int rows, int max_splits) {
    const int stages = W.K / 32;
    const long long tiles = (long long)((W.N / 32 + 7) / 8) * ((rows + 255) / 256);
    int best = 1;
    double best_us = 0;
    for (int s = 1; s <= max(1, min(max_splits, stages / 8)); ++s) {
        const int sps = (stages + s - 1) / s;
        if ((stages + sps - 1) / sps != s) continue;
        const double us = (double)((tiles * s + 255) / 256) * (sps * 0.95 + 8.0) + (double)s * rows * W.N * 8e-6 / 5.0;
        if (best_us == 0 || us < best_us) {
            best_us = us;
            best = s;
        }
    }
    return best;
}

// Column strips of a workgroup, given the split.  A round of 256 workgroups costs 8 us and a stage time for each of its stages.  With
// every unit busy the matrix cores' power bounds a stage: 1.7 us at eight strips, in proportion for fewer; a workgroup alone takes
// 0.95 us however few its strips are (loads and barrier), and a round that is not full lies between the two.  So a partial last round
// costs less than a whole one, but narrower tiles that make whole rounds still win.  Eight strips unless another number promises
// more than a twentieth, which the model is off by itself.  Measured in prefills, eight strips -> picked (us): gate/up of the 8B shape
// at 1024 / 1200 / 1792 rows 412 / 549 / 740 -> 404 / 481 / 706 (seven, six, five), q/k/v at 1024 / 1792 rows 105 / 175 -> 92 / 151 (six);
// the launches beside them, eight strips on both sides, take 2 to 3 % longer (what a launch saves in time it draws in power).  All
// kernels of two layers: 8B shape at 1024 / 1200 / 1792 rows 1987 / 2372 / 3239 -> 1945 / 2274 / 3156, 14B shape at 512 / 1024 rows
// 1450 / 2393 -> 1423 / 2407.  One row tile (a vocabulary above 128 rows) takes eight: no two workgroups share a column's weights there, and
// seven strips, which the figures promise 6 % for, took 664 / 693 us instead of 640 / 674 (152 064 x 5120 at 200 / 256 rows).
static int wide_pick_strips(const Mat& W, int rows, int splits) {
    const int stages = W.K / 32, strips = W.N / 32, row_tiles = (rows + 255) / 256, sps = (stages + splits - 1) / splits;
    if (row_tiles == 1) return 8;
    const auto cost = [&](int cb) {
        const long long wgs = (long long)((strips + cb - 1) / cb) * row_tiles * splits, rounds = (wgs + 255) / 256;
        const double full = (double)wgs / (double)(rounds * 256), stage = 0.95 + (1.7 * cb / 8 - 0.95) * full;
        return (double)rounds * (sps * stage + 8.0);
    };
    int best = 8;
    double best_us = cost(8) * 0.95;
    for (int cb = 7; cb >= 5; --cb)
        if (const double us = cost(cb); us < best_us) {
            best_us = us;
            best = cb;
        }
    return best;
}

// Gate/up: SwiGLU in the epilogue, which needs every sum whole (no split along k), or slabs and a kernel of their own.
// bf16 only (the 4-bit down projection wants its input's group sums).  Above 64 rows the epilogue always wins.  Up to 64
// rows it does where the columns alone nearly fill the chip, from 208 workgroups of four waves on; it saves a launch and
// the slabs.  A layer, hidden 4096, slabs -> epilogue (us), at 1 / 16 / 64 rows: 160 workgroups (ffn 10240) 111 / 117 / 134 ->
// 114 / 119 / 141, 192 (12288) 120 / 126 / 143 -> 118 / 123 / 145, 256 (16384) 134 / 138 / 158 -> 130 / 134 / 153, 448
// (28672) 177 / 185 / 212 -> 175 / 179 / 198; hidden 2048 alike; hidden 5120 with 216 (14B shape): 176 / 193 / 268 -> 177 /
// 191 / 266; 8B shape (224), step of 8 layers: 1167 / 1279 / 1792 -> 1150 / 1243 / 1759.
bool proj_fuses_swiglu(const Mat& gu, int rows) {
    return gu.kind == MAT_BF16_PACKED && (rows > 64 || (gu.N / 32 + 3) / 4 >= 208);
}

int proj_pick_splits(const Mat& W, int rows, int max_splits) {
    if (use_wide(W, rows)) return wide_pick_splits(W, rows, max_splits);
    if (use_tall(W, rows)) return tall_pick_splits(W, rows, max_splits);
    return proj_pick(W, rows, max_splits).splits;
}

static constexpr int waves_by_cost(int strips, int kch, int mtiles, int most, int splits, int ends = 6) {
    int best = 4;
    for (int nw = 5; nw <= most; ++nw)
        if (proj_cost(strips, kch, mtiles, nw, splits, ends) < proj_cost(strips, kch, mtiles, best, splits, ends)) best = nw;
    return best;
}
// The vocabulary (one matrix, never split).  From two rounds of workgroups of seven waves on it is bound otherwise than by starts and ends: every round
// streams beside the last one's end, and what counts is the activation tile that each workgroup stages again, about two strips' worth.
// Waves by starts and ends -> by the tile, us of the projection at 1 / 32 / 64 rows: 128 256 x 256 six -> four 20.6 / 23.7 / 26.5 -> 15.4 / 18.1 / 22.9;
// 152 064 five -> seven x 1024 62.8 / 73.2 / 82.5 -> 58.6 / 70.7 / 78.1, x 4096 212 / 240 / 280 -> 205 / 235 / 251, x 5120 262 / 296 / 346 -> 252 / 288 /
// 307; 256 000 x 2048 four -> seven 188 / 220 / 233 -> 184 / 213 / 225.  128 256 x 4096 (four by either) with five / six / seven is 2 to 20 % slower.
// Up to 32 rows the tile is half as large, and with long k the four that starts and ends ask for stay (two such workgroups share a
// compute unit): 256 000 x 3072 four -> seven 254 / 297 -> 266 / 302 us at 1 / 32 rows (334 -> 321 at 64), x 5120 409 / 468 -> 426 / 473
// (531 -> 502), 262 144 x 5120 417 / 475 -> 427 / 482 (523 -> 510); five stay seven: 320 000 x 3072 326 / 386 -> 320 / 376, x 5120 524 / 617 -> 515 / 602.
// Above 327 680 columns starts and ends choose again: 352 000 four -> five at 64 rows x 2048 319 -> 333, x 4096 609 -> 635.
static constexpr int vocab_waves(int strips, int kch, int rows) {
    const int by_ends = waves_by_cost(strips, kch, 1, 7, 1);
    if (strips < 7 * 512 || strips > 10240 || (rows <= 32 && kch >= 24 && by_ends == 4)) return by_ends;
    return waves_by_cost(strips, kch, 1, 7, 1, 2 * kch);
}
static_assert(vocab_waves(4008, 2, 1) == 4 && vocab_waves(4752, 8, 33) == 7 && vocab_waves(4752, 40, 1) == 7 && vocab_waves(8000, 16, 1) == 7, "by the tile");
static_assert(vocab_waves(3583, 2, 1) == 7 && vocab_waves(8000, 24, 32) == 4 && vocab_waves(8192, 40, 32) == 4 && vocab_waves(11000, 32, 64) == 4, "by starts and ends");
static_assert(vocab_waves(8000, 24, 33) == 7 && vocab_waves(8192, 40, 64) == 7 && vocab_waves(10000, 40, 1) == 7, "the larger tile; not four");

// the wave count that goes with a given split factor
static int proj_pick_waves(const Mat& W, int rows, int splits) {
    const int strips = W.N / 32, kch = W.K / 128;
    const ProjTiling t = proj_tiling(W, rows);
    const int mtiles = t.mtiles;
    if (W.kind == MAT_W4_PACKED && mtiles >= 2) return W.N / 32 >= 512 && mtiles <= 2 ? 7 : 4;
    if (W.vocab && t.mb <= 4) return vocab_waves(strips, kch, rows);
    return waves_by_cost(strips, kch, mtiles, t.mb <= 4 ? 7 : 4, splits);
}

template <int MB, int KS>
static hipError_t launch_proj_nw(const ProjArgs& a, int nw, bool stream, int epilogue, int splits, int mtiles, hipStream_t st) {
    const auto go = [&](auto nwc) {
        constexpr int NW = decltype(nwc)::value;
        return stream ? launch_proj_t<MB, KS, NW, true>(a, epilogue, splits, mtiles, st)
                      : launch_proj_t<MB, KS, NW, false>(a, epilogue, splits, mtiles, st);
    };
    switch (nw) {
    case 4: return go(std::integral_constant<int, 4>{});
    case 5: return go(std::integral_constant<int, 5>{});
    case 6: return go(std::integral_constant<int, 6>{});
    case 7: return go(std::integral_constant<int, 7>{});
    }
    return hipErrorInvalidValue;
}

hipError_t launch_proj(const ProjLaunch& p, hipStream_t st) {
    const Mat& W = *p.W;
    const bool w4 = W.kind == MAT_W4_PACKED;
    if (!w4 && W.kind != MAT_BF16_PACKED) return hipErrorInvalidValue;
    if (p.rows < 1 || p.rows > (w4 ? kMaxBatchTile : kMaxPrefillTile) || W.N % 32 || W.K % 128) return hipErrorInvalidValue;
    const ATile at = atile_for_rows(p.rows);
    ProjArgs a{};
    a.W = (const u32x4*)W.w;
    a.SZ = (const uint32_t*)W.sz;
    a.s_only = W.s_only ? 1 : 0;
    a.A = (const u32x4*)p.A;
    a.qscale = p.qscale;
    a.out = p.out;
    a.rows = p.rows;
    a.N = W.N;
    a.K = W.K;
    a.ldo = p.ldo;
    a.ld_rows = p.ld_rows;
    a.mb_rows = at.MB;
    const int kch = W.K / 128;
    int splits = max(1, p.splits);
    const int cps = chunks_per_split(kch, splits);
    splits = (kch + cps - 1) / cps;
    if (w4 && p.qscale == nullptr) return hipErrorInvalidValue;
    const ProjTiling t = proj_tiling(W, p.rows);
    // Up to 64-row tiles a stage is a whole 128-wide group: three 16 KB stages in LDS for 32-row tiles,
    // two 32 KB stages for 64-row tiles (long stages amortise the workgroup barrier better than a
    // third buffer does); the 128-row bf16 tile has 64-wide stages.
    if (t.mb <= 4) {
        a.n_stages = kch;
        a.stages_per_split = cps;
        const int nw = proj_pick_waves(W, p.rows, splits);
        if (w4) {
            if (p.epilogue != EPI_STORE) return hipErrorInvalidValue;
            return launch_proj_w4(a, nw, splits, t.mtiles, st);
        }
        if (t.mb == 2) return launch_proj_nw<2, 128>(a, nw, W.stream, p.epilogue, splits, t.mtiles, st);
        return launch_proj_nw<4, 128>(a, nw, W.stream, p.epilogue, splits, t.mtiles, st);
    }
    if (use_wide(W, p.rows)) {
        const int want = p.epilogue == EPI_SWIGLU ? 1 : max(1, p.splits);
        const int stg = kch * 4, per = (stg + want - 1) / want;
        a.n_stages = stg;
        a.stages_per_split = per;
        const int real_s = (stg + per - 1) / per;
        return launch_proj_wide(a, p.epilogue, wide_pick_strips(W, p.rows, real_s), real_s, st);
    }
    if (use_tall(W, p.rows)) {
        const int want = p.epilogue == EPI_SWIGLU ? 1 : max(1, p.splits);
        const int stg = kch * 2, per = (stg + want - 1) / want, real_s = (stg + per - 1) / per;
        a.n_stages = stg;
        a.stages_per_split = per;
        return launch_proj_tall(a, p.epilogue, real_s, (at.MB + 3) / 4, st);
    }
    a.n_stages = kch * 2;
    a.stages_per_split = cps * 2;
    return launch_proj_t<8, 64, 4, false>(a, p.epilogue, splits, t.mtiles, st);
}

// ---------------------------------------------------------------------------------
// fp32 path (parity configuration): plain vector-ALU dot products, one wave per column
// ---------------------------------------------------------------------------------

struct F32Mat {
    const float* w[3];
    const uint8_t* q[3];
    const uint16_t* s[3];
    const uint16_t* z[3];
    int rows[3];
    int nsrc, N, K, quant;
    const float* gain;  // not NULL: the input is rmsnorm(x) * gain
    float eps;
};

// Eight sums over the wave at once: three exchanges halve what a lane holds (4 + 2 + 1 values), three more finish the
// one it is left with, instead of six per sum.  Each is summed in the order of wave_sum.  Lane bits 5, 4, 3 name
// the sum a lane ends up with.
template <int O, int C>
__device__ __forceinline__ void wave_fold(float (&v)[8]) {
#pragma unroll
    for (int j = 0; j < C; ++j) {
        if constexpr (O >= 16) {
            swap_rows<O>(v[j], v[j + C]);
            v[j] += v[j + C];
        } else {
            const bool up = threadIdx.x & O;
            const float give = up ? v[j] : v[j + C], keep = up ? v[j + C] : v[j];
            v[j] = keep + lane_xor<O>(give);
        }
    }
}
__device__ __forceinline__ float wave_sum8(float (&v)[8]) {
    wave_fold<32, 4>(v);
    wave_fold<16, 2>(v);
    wave_fold<8, 1>(v);
    float t = v[0] + lane_xor<4>(v[0]);
    t += lane_xor<2>(t);
    return t + lane_xor<1>(t);
}

// the sum of row j's lanes, in lanes 8 j .. 8 j + 7
__device__ __forceinline__ float wave_rows(float (&v)[8]) { return wave_sum8(v); }
__device__ __forceinline__ float wave_rows(float (&v)[2]) {
    const float a = wave_sum(v[0]), b = wave_sum(v[1]);
    return (threadIdx.x & 63) < 8 ? a : b;
}

// Bound by launches and latency (the tiny configuration's matrices are a few hundred KiB), so the step's small work rides
// along: the norm in front (f32_fuses_norm; each wave sums its rows' squares for itself), the residual sum or SwiGLU behind.  The
// loads of UN steps along k are in flight together; the sums keep the order of one step at a time (lane l adds k = l, l + 64,
// ... and the lanes meet in a butterfly), the norm's that of a workgroup with a thread per eight columns.  Tiny
// configuration, 8 requests: 5.3 us a launch against 6.4 of the bare products, and 18 launches a step instead of 29; with the first
// weights and the value that is added to requested in front of the rows 4.0 to 4.9, now 3.2 to 4.6.
// The weights' format is asked for in front of the steps: asked at each weight it left a step's loads waiting for one another.  All weights of a step in
// front of its rows, asked for each, against a weight and its rows in turn, asked for once (us): run of 16 steps 849 -> 779; a step of
// 2 layers, hidden 1024 at 1 / 8 / 64 requests 130 / 147 / 339 -> 84 / 99 / 288, 2048 at 1 / 8 319 / 384 -> 176 / 241, 4096 at 1 / 8 669 / 933 -> 380 / 634 (636 /
// 833 where every weight stood beside its rows); 4-bit, hidden 2048 at 1 / 8 / 64 336 / 480 / 1454 -> 236 / 316 / 998.
// BT rows a wave: 8 or 2 (f32_two_rows; the sums are the same ones).
template <int BT, int UN, bool NORM, int EPI>
__global__ __launch_bounds__(256) void proj_f32_kernel(F32Mat m, const float* __restrict__ x, int nrows, float* out) {
    static_assert(BT == 8 || BT == 2, "wave_rows");
    constexpr int NC = EPI == F32_SWIGLU ? 2 : 1;  // columns of a wave: gate and up
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int n = blockIdx.x * 4 + wave, n_out = EPI == F32_SWIGLU ? m.rows[0] : m.N;
    if (n >= n_out) return;
    const int b0 = blockIdx.y * BT, K = m.K;
    int src[NC], r[NC];
    src[0] = 0;
    r[0] = n;
    if constexpr (EPI == F32_SWIGLU) {
        src[1] = 1;
        r[1] = n;
    } else {
        while (src[0] + 1 < m.nsrc && r[0] >= m.rows[src[0]]) {
            r[0] -= m.rows[src[0]];
            ++src[0];
        }
    }
    const float* row[BT];
#pragma unroll
    for (int j = 0; j < BT; ++j) row[j] = x + (size_t)min(b0 + j, nrows - 1) * K;
    const int ng = K / kGroup;
    float wv[UN][NC], gv[UN];
    const auto load_w = [&](auto quant, int i, int at) {
        const int k = min(at, K - 1);  // past the end: valid, not added
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if constexpr (quant) {
                const uint8_t byte = m.q[src[c]][(size_t)r[c] * (K / 2) + (k >> 1)];
                const float code = (float)((k & 1) ? (byte >> 4) : (byte & 15));
                const size_t g = (size_t)r[c] * ng + k / kGroup;
                const float zf = m.z[src[c]] ? __half2float(__ushort_as_half(m.z[src[c]][g])) : 8.f;
                const float sf = __half2float(__ushort_as_half(m.s[src[c]][g]));
                wv[i][c] = (code - zf) * sf;  // exact: 5-bit integer times an 11-bit significand
            } else {
                wv[i][c] = m.w[src[c]][(size_t)r[c] * K + k];
            }
        }
        if constexpr (NORM) gv[i] = m.gain[k];
    };
    const auto first = [&](auto quant) {
#pragma unroll
        for (int i = 0; i < UN; ++i) load_w(quant, i, lane + i * 64);
    };
    // what does not wait for the rows is requested in front of them: the first weights and the value that is added to
    if (m.quant) first(std::true_type{});
    else first(std::false_type{});
    const int b = b0 + (lane >> 3);
    const bool mine = lane < BT * 8 && (lane & 7) == 0 && b < nrows;
    float* o = out + (size_t)min(b, nrows - 1) * n_out + n;
    float before = 0.f;
    if constexpr (EPI == F32_ADD) before = *o;
    float rinv[BT];
    if constexpr (NORM) {  // the rows' sums of squares: eight columns a lane, 512 a round, a round's sum as one wave of a workgroup
        float tot = 0.f;
        for (int u0 = 0; u0 < K / 8; u0 += 64) {
            float ss[BT];
#pragma unroll
            for (int j = 0; j < BT; ++j) {
                ss[j] = 0.f;
                if (u0 + lane < K / 8) {
                    const float* p = row[j] + (size_t)(u0 + lane) * 8;
#pragma unroll
                    for (int e = 0; e < 8; ++e) ss[j] = fmaf(p[e], p[e], ss[j]);
                }
            }
            tot += wave_rows(ss);
        }
        const float ri = 1.0f / sqrtf(tot / (float)K + m.eps);
#pragma unroll
        for (int j = 0; j < BT; ++j) rinv[j] = __shfl(ri, j * 8);
    }
    float acc[NC][BT];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int j = 0; j < BT; ++j) acc[c][j] = 0.f;
    const auto add_up = [&](auto quant) {
        for (int k0 = lane; k0 < K; k0 += 64 * UN) {
            float xv[UN][BT];
#pragma unroll
            for (int i = 0; i < UN; ++i) {
                if (k0 >= 64 * UN) load_w(quant, i, k0 + i * 64);
#pragma unroll
                for (int j = 0; j < BT; ++j) xv[i][j] = row[j][min(k0 + i * 64, K - 1)];
            }
#pragma unroll
            for (int i = 0; i < UN; ++i)
                if (k0 + i * 64 < K) {
#pragma unroll
                    for (int j = 0; j < BT; ++j) {
                        float y = xv[i][j];
                        if constexpr (NORM) y = y * rinv[j] * gv[i];
#pragma unroll
                        for (int c = 0; c < NC; ++c) acc[c][j] = fmaf(wv[i][c], y, acc[c][j]);
                    }
                }
        }
    };
    if (m.quant) add_up(std::true_type{});
    else add_up(std::false_type{});
    float v[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) v[c] = wave_rows(acc[c]);
    if (!mine) return;
    if constexpr (EPI == F32_SWIGLU) *o = v[0] / (1.0f + expf(-v[0])) * v[1];
    else if constexpr (EPI == F32_ADD) *o = before + v[0];
    else *o = v[0];
}

static int f32_out_cols(const Mat& W, int epilogue) { return epilogue == F32_SWIGLU ? W.src_rows[0] : W.N; }

// The norm rides along as long as summing each row's squares in every wave costs less than the launch it saves, about 4 us.
// Step of 4 layers, inside / launch of its own (us): hidden 256, ffn 688 at 1 / 8 / 32 / 64 / 128 rows 81 / 102 / 121 / 149 / 189 against
// 115 / 121 / 127 / 141 / 164, hidden 512, ffn 1024 at 8 / 32 / 64 rows 115 / 175 / 236 against 129 / 168 / 211, hidden 1024, ffn 2816 at
// 1 / 4 / 8 / 64 rows 150 / 163 / 200 / 687 against 152 / 163 / 176 / 515, hidden 2048 at 256 rows 8.4 ms against 5.7.  Above 8192 columns the norm
// kernel sums in another order than a wave does here.
bool f32_fuses_norm(const Mat& W, int rows, int epilogue) {
    return W.K <= 8192 && (long long)f32_out_cols(W, epilogue) * rows * W.K <= (W.K <= 512 ? 1 << 24 : 1 << 23);
}

// Two rows a wave, or eight: two where eight would leave most of the chip without a workgroup (eight workgroups fit a compute
// unit), as long as the matrix, which every group of rows reads again, is not the larger cost.  Down projection, two / eight
// rows a wave (us): 1024 x 2816 at 1 / 8 / 16 rows 7.0 / 7.1 / 11.2 against 8.7 / 8.3 / 11.9, 2048 x 2048 (O) at 1 / 4 / 8 rows 7.1 /
// 7.1 / 9.0 against 8.1 / 7.9 / 8.0, 2048 x 6144 at 1 / 8 rows 14 / 24 against 24 / 24, 4096 x 14336 at 1 / 4 / 6 / 8 rows 36 / 68 / 100 / 132 against
// 71 / 70 / 71 / 80.
static bool f32_two_rows(const Mat& W, int cols, int rows) {
    const int groups = (rows + 1) / 2;
    return groups == 1 || (long long)cols * groups <= (groups == 2 || W.K >= 4096 ? 2048 : 1024);
}

hipError_t launch_proj_f32(const Mat& W, const float* x, int rows, const void* gain, float eps, int epilogue, float* out, hipStream_t st) {
    F32Mat m{};
    m.nsrc = W.nsrc;
    m.N = W.N;
    m.K = W.K;
    m.quant = W.kind == MAT_W4_LOGICAL;
    m.gain = (const float*)gain;
    m.eps = eps;
    if (!m.quant && W.kind != MAT_F32) return hipErrorInvalidValue;
    for (int i = 0; i < 3; ++i) {
        m.w[i] = (const float*)W.wsrc[i];
        m.q[i] = W.q[i];
        m.s[i] = W.s[i];
        m.z[i] = W.z[i];
        m.rows[i] = W.src_rows[i];
    }
    if (gain && W.K % 8) return hipErrorInvalidValue;
    if (epilogue == F32_SWIGLU && (W.nsrc != 2 || m.rows[0] != m.rows[1])) return hipErrorInvalidValue;
    const int cols = (f32_out_cols(W, epilogue) + 3) / 4;
    const auto go = [&](auto bt, auto un) {
        constexpr int BT = decltype(bt)::value, UN = decltype(un)::value;
        const dim3 grid(cols, (rows + BT - 1) / BT), block(256);
        if (gain) {
            switch (epilogue) {
            case F32_STORE: hipLaunchKernelGGL((proj_f32_kernel<BT, UN, true, F32_STORE>), grid, block, 0, st, m, x, rows, out); break;
            case F32_SWIGLU: hipLaunchKernelGGL((proj_f32_kernel<BT, UN, true, F32_SWIGLU>), grid, block, 0, st, m, x, rows, out); break;
            default: return hipErrorInvalidValue;
            }
        } else {
            switch (epilogue) {
            case F32_STORE: hipLaunchKernelGGL((proj_f32_kernel<BT, UN, false, F32_STORE>), grid, block, 0, st, m, x, rows, out); break;
            case F32_ADD: hipLaunchKernelGGL((proj_f32_kernel<BT, UN, false, F32_ADD>), grid, block, 0, st, m, x, rows, out); break;
            case F32_SWIGLU: hipLaunchKernelGGL((proj_f32_kernel<BT, UN, false, F32_SWIGLU>), grid, block, 0, st, m, x, rows, out); break;
            default: return hipErrorInvalidValue;
            }
        }
        return hipGetLastError();
    };
    // steps of 64 along k in flight: four for one group of rows (2048 x 6144 at 8 rows 24 us, one step 39), one where several
    // groups of waves cover each other's waits (at 16 / 24 / 32 / 64 / 256 rows 40 / 47 / 68 / 123 / 479 us, four steps 32 / 51 / 62 / 125 / 492)
    if (f32_two_rows(W, cols, rows)) return go(std::integral_constant<int, 2>{}, std::integral_constant<int, 4>{});
    if (rows <= 8) return go(std::integral_constant<int, 8>{}, std::integral_constant<int, 4>{});
    return go(std::integral_constant<int, 8>{}, std::integral_constant<int, 1>{});
}

// ---------------------------------------------------------------------------------
// packing
// ---------------------------------------------------------------------------------

size_t packed_bf16_bytes(int N, int K) { return (size_t)N * K * 2; }
size_t packed_w4_bytes(int N, int K) { return (size_t)N * K / 2; }
size_t packed_w4_sz_bytes(int N, int K) { return (size_t)N * (K / 128) * 4; }

struct PackSrc {
    const void* p[3];
    const void* s[3];
    const void* z[3];
    int rows[3];
    int nsrc, mode, K, N;
};

// packed row pn -> (source, row).  mode 0: stacked.  mode 1: blocks of 16 rows alternate
// between source 0 (gate) and source 1 (up).
__device__ __forceinline__ void pack_row(const PackSrc& s, int pn, int& src, int& row) {
    if (s.mode == 1) {
        src = (pn >> 4) & 1;
        row = (pn >> 5) * 16 + (pn & 15);
    } else {
        src = 0;
        row = pn;
        while (src + 1 < s.nsrc && row >= s.rows[src]) {
            row -= s.rows[src];
            ++src;
        }
    }
}

// one thread per 16-byte unit of the packed matrix: [N/32][K/128][8][64] x 8 bf16
__global__ __launch_bounds__(256) void pack_bf16_kernel(PackSrc s, u32x4* __restrict__ dst) {
    const size_t u = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t total = (size_t)s.N * s.K / 8;
    if (u >= total) return;
    const int lane = (int)(u & 63), kk = (int)((u >> 6) & 7);
    const size_t t = u >> 9;
    const int kch = s.K / 128;
    const int c = (int)(t % kch), nb = (int)(t / kch);
    const int pn = nb * 32 + (lane & 31), half = lane >> 5;
    const int k = c * 128 + half * 64 + kk * 8;
    int src, row;
    pack_row(s, pn, src, row);
    dst[u] = *reinterpret_cast<const u32x4*>((const uint16_t*)s.p[src] + (size_t)row * s.K + k);
}

// one thread per packed dword (8 codes): [N/32][K/128][2][64][4 dwords]
__global__ __launch_bounds__(256) void pack_w4_kernel(PackSrc s, uint32_t* __restrict__ dst,
                                                      uint32_t* __restrict__ dst_sz) {
    const size_t u = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t total = (size_t)s.N * s.K / 8;
    if (u >= total) return;
    const int comp = (int)(u & 3), lane = (int)((u >> 2) & 63), j = (int)((u >> 8) & 1);
    const size_t t = u >> 9;
    const int kch = s.K / 128;
    const int c = (int)(t % kch), nb = (int)(t / kch);
    const int kk = j * 4 + comp;
    const int pn = nb * 32 + (lane & 31), half = lane >> 5;
    const int k = c * 128 + half * 64 + kk * 8;
    int src, row;
    pack_row(s, pn, src, row);
    const uint32_t word = *reinterpret_cast<const uint32_t*>((const uint8_t*)s.p[src] + ((size_t)row * s.K + k) / 2);
    // logical: code e at bits [4e, 4e+4).  packed: the low nibbles of the four bytes hold e = 0..3, the
    // high nibbles e = 4..7, so that "and 0x0F0F0F0F" and "shift by 4, and" give the codes as bytes in order
    uint32_t o = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) o |= ((word >> (4 * e)) & 15u) << (e < 4 ? 8 * e : 8 * (e - 4) + 4);
    dst[u] = o;
    if (kk == 0 && half == 0) {
        const size_t g = (size_t)row * kch + c;
        const uint32_t sv = ((const uint16_t*)s.s[src])[g];
        if (s.z[src]) {
            const uint32_t zv = ((const uint16_t*)s.z[src])[g];
            dst_sz[((size_t)nb * kch + c) * 32 + (lane & 31)] = sv | (zv << 16);
        } else {  // scales only: groups 2i and 2i+1 share a dword
            ((uint16_t*)dst_sz)[(((size_t)nb * ((kch + 1) >> 1) + (c >> 1)) * 32 + (lane & 31)) * 2 + (c & 1)] = (uint16_t)sv;
        }
    }
}

static PackSrc make_src(const void* const p[3], const void* const s[3], const void* const z[3],
                        const int rows[3], int nsrc, int mode, int K) {
    PackSrc ps{};
    ps.nsrc = nsrc;
    ps.mode = mode;
    ps.K = K;
    ps.N = 0;
    for (int i = 0; i < 3; ++i) {
        ps.p[i] = p[i];
        ps.s[i] = s ? s[i] : nullptr;
        ps.z[i] = z ? z[i] : nullptr;
        ps.rows[i] = i < nsrc ? rows[i] : 0;
        ps.N += ps.rows[i];
    }
    return ps;
}

hipError_t launch_pack_bf16(const void* const src[3], const int src_rows[3], int nsrc, int mode, int K, void* dst,
                            hipStream_t st) {
    PackSrc ps = make_src(src, nullptr, nullptr, src_rows, nsrc, mode, K);
    const size_t total = (size_t)ps.N * K / 8;
    hipLaunchKernelGGL(pack_bf16_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, ps, (u32x4*)dst);
    return hipGetLastError();
}

hipError_t launch_pack_w4(const sun_qmat src[3], const int src_rows[3], int nsrc, int mode, int K, void* dst_codes,
                          void* dst_sz, hipStream_t st) {
    const void *p[3] = {nullptr, nullptr, nullptr}, *s[3] = {nullptr, nullptr, nullptr}, *z[3] = {nullptr, nullptr, nullptr};
    for (int i = 0; i < nsrc; ++i) {
        p[i] = src[i].q;
        s[i] = src[i].s;
        z[i] = src[i].z;
    }
    PackSrc ps = make_src(p, s, z, src_rows, nsrc, mode, K);
    const size_t total = (size_t)ps.N * K / 8;
    hipLaunchKernelGGL(pack_w4_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, ps,
                       (uint32_t*)dst_codes, (uint32_t*)dst_sz);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// round-to-nearest group quantiser (one wave per group of 128 weights)
// ---------------------------------------------------------------------------------

__global__ __launch_bounds__(256) void quantize_w4_kernel(const void* __restrict__ w, int dtype, int rows, int cols,
                                                          int mode, uint8_t* __restrict__ q, uint16_t* __restrict__ s,
                                                          uint16_t* __restrict__ z) {
    const int lane = threadIdx.x & 63;
    const size_t grp = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int ng = cols / kGroup;
    if (grp >= (size_t)rows * ng) return;
    const size_t row = grp / ng;
    const int g = (int)(grp % ng);
    const size_t e0 = row * cols + (size_t)g * kGroup + 2 * lane;
    float a, b;
    if (dtype == SUN_BF16) {
        const uint32_t pr = *reinterpret_cast<const uint32_t*>((const uint16_t*)w + e0);
        a = bf16_lo(pr);
        b = bf16_hi(pr);
    } else {
        a = ((const float*)w)[e0];
        b = ((const float*)w)[e0 + 1];
    }
    const float mn = -wave_max(-fminf(a, b)), mx = wave_max(fmaxf(a, b));
    const float amax = wave_max(fmaxf(fabsf(a), fabsf(b)));
    const float sf = mode == 0 ? __fdiv_rn(mx - mn, 15.0f) : __fdiv_rn(amax, 7.0f);
    __half sh = __float2half_rn(sf);
    float S = __half2float(sh);
    if (S == 0.f) {
        S = 1.f;
        sh = __float2half_rn(1.f);
    }
    const float Z = mode == 0 ? fminf(fmaxf(rintf(__fdiv_rn(-mn, S)), 0.f), 15.f) : 8.f;
    const int qa = (int)fminf(fmaxf(rintf(__fdiv_rn(a, S)) + Z, 0.f), 15.f);
    const int qb = (int)fminf(fmaxf(rintf(__fdiv_rn(b, S)) + Z, 0.f), 15.f);
    q[(row * cols + (size_t)g * kGroup) / 2 + lane] = (uint8_t)(qa | (qb << 4));
    if (lane == 0) {
        s[grp] = __half_as_ushort(sh);
        if (z) z[grp] = __half_as_ushort(__float2half_rn(Z));
    }
}

hipError_t launch_quantize_w4(const void* w, int dtype, int rows, int cols, int group, int mode, void* q, void* s,
                              void* z, hipStream_t st) {
    if (group != kGroup || cols % kGroup) return hipErrorInvalidValue;
    const size_t groups = (size_t)rows * (cols / kGroup);
    hipLaunchKernelGGL(quantize_w4_kernel, dim3((unsigned)((groups + 3) / 4)), dim3(256), 0, st, w, dtype, rows, cols,
                       mode, (uint8_t*)q, (uint16_t*)s, (uint16_t*)z);
    return hipGetLastError();
}

}  // namespace sun
