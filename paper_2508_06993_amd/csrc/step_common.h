// Device building blocks shared by the matrix-core step kernels: vector types,
// MLP policies (operand precision), fire-bit ballots, storage chunks and
// buffer descriptors.  Internal header, included by the kernel files only.
#pragma once

#include "device_common.h"

namespace octnca {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v8f __attribute__((ext_vector_type(8)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));

// Feature order seen by lane (g, n): slot s < 4 is state channel 4g + s,
// slot s >= 4 is perception channel 4g + s - 4.
__device__ __forceinline__ int feature_of(int slot, int g) {
    return slot < 4 ? 4 * g + slot : kC + 4 * g + (slot - 4);
}

// Marks a register value as produced here (an empty asm that reads and
// rewrites it): loads of kernel-wide constants then complete in the prologue
// instead of being sunk into the tile loop, where the compiler would have to
// wait for all outstanding memory operations at their first use.
template <typename V>
__device__ __forceinline__ void pin(V &x) {
    asm volatile("" : "+v"(x));
}

// ---------------------------------------------------------------------------
// MLP policies.  Each gathers its weights into lane registers once per block
// (load) and computes the update of channels 4g..4g+3 of the lane's cell from
// its 8 features in two halves: layer1 (features -> hidden accumulators, all
// MFMA) and layer2 (ReLU, hidden -> update).  Splitting them lets a wave
// issue the next group's perception while layer 1's MFMAs run.  All
// accumulate in fp32.  The second layer has outputs for the hidden channels
// only (Sec. 3.1): load() gathers the W2 rows of the nin input channels as
// zeros, so their update is exactly +0 and the residual needs no per-channel
// mask.  ld1 / ld2: floats between W1's and W2's rows (padded copies in LDS).
// Those rows are loaded like the others and then replaced by zero: a
// load behind the lane condition became a branch and a full memory wait per
// element (16 round trips, about 5 us per launch, measured).
// kPerceptionScale: the factor the kernel applies to the perception weights
// and bias (features 4..7 arrive multiplied by it).
// kSelectGate: how the fire gate is applied (gated() below).
// ---------------------------------------------------------------------------

// ReLU as an integer max on the float's bits: negative floats (sign bit set)
// are negative integers and become +0; one instruction, no NaN quieting.
__device__ __forceinline__ float relu(float x) {
    return __int_as_float(max(__float_as_int(x), 0));
}

// fp32 operands: v_mfma_f32_16x16x4_f32, 32 + 16 MFMAs per 16 cells.
struct MlpF32 {
    static constexpr int kChannels = kC, kHidden = kH;
    static constexpr float kPerceptionScale = 1.f;
    static constexpr bool kSelectGate = false;
    float w1[4][8];   // [jt][kc] = W1[jt*16 + n][feature(kc, g)]
    v4f b1[4];        // [jt][i]  = b1[jt*16 + 4g + i]
    float w2[4][4];   // [jt][i]  = W2[n][jt*16 + 4g + i]   (n = output channel)

    __device__ __forceinline__ void pin_all() {
#pragma unroll
        for (int jt = 0; jt < 4; ++jt) {
#pragma unroll
            for (int k = 0; k < 8; ++k) pin(w1[jt][k]);
#pragma unroll
            for (int i = 0; i < 4; ++i) pin(w2[jt][i]);
            pin(b1[jt]);
        }
    }

    __device__ __forceinline__ void load(const float *__restrict__ W1, const float *__restrict__ B1,
                                         const float *__restrict__ W2, int n, int g, int nin,
                                         int ld1 = 2 * kChannels, int ld2 = kHidden) {
#pragma unroll
        for (int jt = 0; jt < 4; ++jt) {
#pragma unroll
            for (int kc = 0; kc < 8; ++kc) w1[jt][kc] = W1[(jt * 16 + n) * ld1 + feature_of(kc, g)];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                b1[jt][i] = B1[jt * 16 + 4 * g + i];
                const float v = W2[n * ld2 + jt * 16 + 4 * g + i];   // loaded for every n
                w2[jt][i] = n < nin ? 0.f : v;
            }
        }
    }

    __device__ __forceinline__ void layer1(const float f[8], v4f acc[4]) const {
#pragma unroll
        for (int jt = 0; jt < 4; ++jt)
            acc[jt] = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[jt][0], f[0], b1[jt], 0, 0, 0);
#pragma unroll
        for (int kc = 1; kc < 8; ++kc)
#pragma unroll
            for (int jt = 0; jt < 4; ++jt)
                acc[jt] = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[jt][kc], f[kc], acc[jt], 0, 0, 0);
    }

    __device__ __forceinline__ v4f layer2(const v4f acc[4]) const {
        v4f u0 = {0.f, 0.f, 0.f, 0.f}, u1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int jt = 0; jt < 4; ++jt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float h = relu(acc[jt][i]);
                if ((jt * 4 + i) & 1)
                    u1 = __builtin_amdgcn_mfma_f32_16x16x4f32(w2[jt][i], h, u1, 0, 0, 0);
                else
                    u0 = __builtin_amdgcn_mfma_f32_16x16x4f32(w2[jt][i], h, u0, 0, 0, 0);
            }
        return u0 + u1;
    }
};

// Split-precision bf16: every fp32 operand x is written as hi + lo with
// hi = bf16(x), lo = bf16(x - hi); a product a*b is taken as
// hi_a*hi_b + hi_a*lo_b + lo_a*hi_b (the dropped lo*lo term is below 2^-16
// relative), on v_mfma_f32_16x16x32_bf16 with fp32 accumulation.  The K = 32
// operand of a lane is 8 consecutive K slots, so one MFMA covers all 32
// features of layer 1 and two cover the 64 hidden units of layer 2:
// 12 + 6 MFMAs per 16 cells.  A and B use the same (lane group, slot) -> K
// correspondence, so the feature / hidden order only has to agree between
// the weights gathered here and the activations.
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));

// hi = bf16(x) (round to nearest even, two values per conversion), hi read
// back as fp32 by bit shifts, lo = bf16(x - hi).
__device__ __forceinline__ void split_bf16(const v8f &x, v8bf &hi, v8bf &lo) {
    uint32_t h[4], l[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const v2bf hp = __builtin_convertvector(v2f{x[2 * p], x[2 * p + 1]}, v2bf);
        h[p] = __builtin_bit_cast(uint32_t, hp);
        const float back0 = __uint_as_float(h[p] << 16);
        const float back1 = __uint_as_float(h[p] & 0xffff0000u);
        const v2bf lp = __builtin_convertvector(v2f{x[2 * p] - back0, x[2 * p + 1] - back1}, v2bf);
        l[p] = __builtin_bit_cast(uint32_t, lp);
    }
    hi = __builtin_bit_cast(v8bf, h);
    lo = __builtin_bit_cast(v8bf, l);
}

struct MlpBf16x3 {
    static constexpr int kChannels = kC, kHidden = kH;
    static constexpr float kPerceptionScale = 1.f;
    static constexpr bool kSelectGate = false;
    v8bf w1h[4], w1l[4];   // [jt] slot s: W1[jt*16 + n][feature(s, g)]
    v4f b1[4];
    v8bf w2h[2], w2l[2];   // [p] slot s: W2[n][hidden(p, s, g)]

    __device__ __forceinline__ void pin_all() {
#pragma unroll
        for (int jt = 0; jt < 4; ++jt) {
            pin(w1h[jt]);
            pin(w1l[jt]);
            pin(b1[jt]);
        }
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            pin(w2h[p]);
            pin(w2l[p]);
        }
    }

    // hidden unit in K slot s of layer-2 MFMA p for lane group g: it is the
    // layer-1 accumulator register (jt = 2p + s/4, i = s%4) of the lane.
    __device__ static __forceinline__ int hidden_of(int p, int s, int g) {
        return (2 * p + s / 4) * 16 + 4 * g + (s % 4);
    }

    __device__ __forceinline__ void load(const float *__restrict__ W1, const float *__restrict__ B1,
                                         const float *__restrict__ W2, int n, int g, int nin,
                                         int ld1 = 2 * kChannels, int ld2 = kHidden) {
#pragma unroll
        for (int jt = 0; jt < 4; ++jt) {
            v8f x;
#pragma unroll
            for (int s = 0; s < 8; ++s) x[s] = W1[(jt * 16 + n) * ld1 + feature_of(s, g)];
            split_bf16(x, w1h[jt], w1l[jt]);
#pragma unroll
            for (int i = 0; i < 4; ++i) b1[jt][i] = B1[jt * 16 + 4 * g + i];
        }
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            v8f x;
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const float v = W2[n * ld2 + hidden_of(p, s, g)];   // loaded for every n
                x[s] = n < nin ? 0.f : v;
            }
            split_bf16(x, w2h[p], w2l[p]);
        }
    }

    __device__ __forceinline__ void layer1(const float f[8], v4f acc[4]) const {
        v8f fx;
#pragma unroll
        for (int s = 0; s < 8; ++s) fx[s] = f[s];
        v8bf fh, fl;
        split_bf16(fx, fh, fl);
#pragma unroll
        for (int jt = 0; jt < 4; ++jt)
            acc[jt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1l[jt], fh, b1[jt], 0, 0, 0);
#pragma unroll
        for (int jt = 0; jt < 4; ++jt)
            acc[jt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1h[jt], fl, acc[jt], 0, 0, 0);
#pragma unroll
        for (int jt = 0; jt < 4; ++jt)
            acc[jt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1h[jt], fh, acc[jt], 0, 0, 0);
    }

    __device__ __forceinline__ v4f layer2(const v4f acc[4]) const {
        v8bf hh[2], hl[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            v8f x;
#pragma unroll
            for (int s = 0; s < 8; ++s) x[s] = relu(acc[2 * p + s / 4][s % 4]);
            split_bf16(x, hh[p], hl[p]);
        }
        v4f u[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            u[p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2l[p], hh[p], v4f{0.f, 0.f, 0.f, 0.f},
                                                           0, 0, 0);
            u[p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2h[p], hl[p], u[p], 0, 0, 0);
        }
#pragma unroll
        for (int p = 0; p < 2; ++p)
            u[p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2h[p], hh[p], u[p], 0, 0, 0);
        return u[0] + u[1];
    }
};

// Feature order of a model with C channels (C <= 16, a multiple of 4): slot
// s < 4 of lane group g is state channel 4g + s, slot s >= 4 perception
// channel 4g + s - 4; lane groups g >= C / 4 hold no channel.
template <int C>
__device__ __forceinline__ int feature_of_c(int slot, int g) {
    return slot < 4 ? 4 * g + slot : C + 4 * g + (slot - 4);
}

// fp16 operands, single pass (for fp16 state storage): weights, features and
// hidden activations rounded to fp16, products accumulated in fp32 on
// v_mfma_f32_16x16x32_f16; 4 + 2 MFMAs per 16 cells.
template <int C, int H>
struct MlpF16M {
    static_assert(C % 4 == 0 && C <= kC && H % 16 == 0 && H <= kH, "fits the 16 / 64 lanes");
    static constexpr int kChannels = C, kHidden = H;
    static constexpr int NT = H / 16;   // hidden tiles computed (a smaller model: see MlpF16SM)
    static constexpr float kPerceptionScale = 1.f;
    // 12 / 48: a cell that does not fire keeps its stored bits whatever its
    // update is, and a sum is rounded to fp32 and then to fp16, as on the generic
    // kernel, which serves this model's other layout (the fma and the conversion
    // became one mixed-precision fma, with one rounding)
    static constexpr bool kSelectGate = C != kC;
    v8h w1[NT];
    v4f b1[NT];
    v8h w2[2];

    __device__ __forceinline__ void pin_all() {
#pragma unroll
        for (int jt = 0; jt < NT; ++jt) {
            pin(w1[jt]);
            pin(b1[jt]);
        }
        pin(w2[0]);
        pin(w2[1]);
    }

    __device__ __forceinline__ void load(const float *__restrict__ W1, const float *__restrict__ B1,
                                         const float *__restrict__ W2, int n, int g, int nin,
                                         int ld1 = 2 * kChannels, int ld2 = kHidden) {
        const bool g_ok = g < C / 4;
        const int gc = g_ok ? g : 0;
#pragma unroll
        for (int jt = 0; jt < NT; ++jt) {
            v8f x;
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const float v = W1[(jt * 16 + n) * ld1 + feature_of_c<C>(s, gc)];
                x[s] = g_ok ? v : 0.f;
            }
            w1[jt] = __builtin_convertvector(x, v8h);
#pragma unroll
            for (int i = 0; i < 4; ++i) b1[jt][i] = B1[jt * 16 + 4 * g + i];
        }
        const bool row_ok = n >= nin && n < C;
        const int nc = n < C ? n : 0;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            v8f x;
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int hid = MlpBf16x3::hidden_of(p, s, g);
                const float v = W2[nc * ld2 + (hid < H ? hid : 0)];   // loaded for every n
                x[s] = row_ok && hid < H ? v : 0.f;
            }
            w2[p] = __builtin_convertvector(x, v8h);
        }
    }

    __device__ __forceinline__ void layer1(const float f[8], v4f acc[4]) const {
        v8f fx;
#pragma unroll
        for (int s = 0; s < 8; ++s) fx[s] = f[s];
        layer1_h(__builtin_convertvector(fx, v8h), acc);
    }

    // features already in fp16 (slot s = feature_of(s, g))
    __device__ __forceinline__ void layer1_h(const v8h &fh, v4f acc[4]) const {
#pragma unroll
        for (int jt = 0; jt < NT; ++jt)
            acc[jt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w1[jt], fh, b1[jt], 0, 0, 0);
    }

    // ReLU after the rounding to fp16, as packed fp16 max (half the
    // instructions of an fp32 max; rounding is monotonic and keeps 0, so the
    // operand is the same fp16 value).  Hidden tiles that are not computed
    // enter as zeros.
    __device__ __forceinline__ v4f layer2(const v4f acc[4]) const {
        v4f u = {0.f, 0.f, 0.f, 0.f};
        const v8h zero = {};
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            v8f x;
#pragma unroll
            for (int s = 0; s < 8; ++s) x[s] = 2 * p + s / 4 < NT ? acc[2 * p + s / 4][s % 4] : 0.f;
            const v8h h = __builtin_elementwise_max(__builtin_convertvector(x, v8h), zero);
            u = __builtin_amdgcn_mfma_f32_16x16x32_f16(w2[p], h, u, 0, 0, 0);
        }
        return u;
    }
};
using MlpF16 = MlpF16M<kC, kH>;

// Scaled fp16 activations with split fp16 weights (for fp32 states).  The
// features and the hidden units are rounded to fp16 after a scaling by 2^-8
// (a power of two: exact), which keeps fp32 states of magnitude up to
// 65504 * 2^8 in fp16 range; the weights are hi + lo fp16 pairs (W1 as is,
// b1 times 2^-8 as the accumulator start, W2 times 2^8 so that u comes out
// unscaled), two products per weight: 8 + 4 MFMAs per 16 cells and no
// activation split.  The activations keep fp16's 2^-12 relative rounding,
// the weights about 2^-22.
constexpr float kF16ActScale = 1.f / 256.f;

// C / H: the model's size.  The lane layout is that of C = 16, H = 64; a
// smaller model (C = 12, H = 48 of the paper's ablation, supplement S10)
// leaves channel quad 3 and hidden tile 3 empty.  Their weights are gathered
// as zeros (loaded from clamped indices and then replaced), hidden tile 3 is
// not computed, and the update of channels >= C is +0.
template <int C, int H>
struct MlpF16SM {
    static_assert(C % 4 == 0 && C <= kC && H % 16 == 0 && H <= kH, "fits the 16 / 64 lanes");
    static constexpr int kChannels = C, kHidden = H;
    static constexpr int NT = H / 16;   // hidden tiles computed
    static constexpr float kPerceptionScale = kF16ActScale;
    static constexpr bool kSelectGate = false;
    v8h w1h[NT], w1l[NT];   // [jt] slot s: W1[jt*16 + n][feature(s, g)], hi + lo
    v4f b1[NT];             // b1 * 2^-8
    v8h w2h[2], w2l[2];     // [p] slot s: 2^8 W2[n][hidden(p, s, g)], hi + lo

    __device__ __forceinline__ void pin_all() {
#pragma unroll
        for (int jt = 0; jt < NT; ++jt) {
            pin(w1h[jt]);
            pin(w1l[jt]);
            pin(b1[jt]);
        }
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            pin(w2h[p]);
            pin(w2l[p]);
        }
    }

    __device__ static __forceinline__ void split(const v8f &x, v8h &hi, v8h &lo) {
        hi = __builtin_convertvector(x, v8h);
        lo = __builtin_convertvector(x - __builtin_convertvector(hi, v8f), v8h);
    }

    __device__ __forceinline__ void load(const float *__restrict__ W1, const float *__restrict__ B1,
                                         const float *__restrict__ W2, int n, int g, int nin,
                                         int ld1 = 2 * kChannels, int ld2 = kHidden) {
        const bool g_ok = g < C / 4;
        const int gc = g_ok ? g : 0;
#pragma unroll
        for (int jt = 0; jt < NT; ++jt) {
            v8f x;
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const float v = W1[(jt * 16 + n) * ld1 + feature_of_c<C>(s, gc)];
                x[s] = g_ok ? v : 0.f;
            }
            split(x, w1h[jt], w1l[jt]);
#pragma unroll
            for (int i = 0; i < 4; ++i) b1[jt][i] = B1[jt * 16 + 4 * g + i] * kF16ActScale;
        }
        // rows of the input channels and of channels >= C are zero
        const bool row_ok = n >= nin && n < C;
        const int nc = n < C ? n : 0;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            v8f x;
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int hid = MlpBf16x3::hidden_of(p, s, g);
                const float v = W2[nc * ld2 + (hid < H ? hid : 0)];   // loaded for every n
                x[s] = row_ok && hid < H ? v * (1.f / kF16ActScale) : 0.f;
            }
            split(x, w2h[p], w2l[p]);
        }
    }

    __device__ __forceinline__ void layer1(const float f[8], v4f acc[4]) const {
        v8f fx;   // state features scaled here, the perception arrives scaled
#pragma unroll
        for (int s = 0; s < 8; ++s) fx[s] = s < 4 ? f[s] * kF16ActScale : f[s];
        const v8h fh = __builtin_convertvector(fx, v8h);
#pragma unroll
        for (int jt = 0; jt < NT; ++jt)
            acc[jt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w1l[jt], fh, b1[jt], 0, 0, 0);
#pragma unroll
        for (int jt = 0; jt < NT; ++jt)
            acc[jt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w1h[jt], fh, acc[jt], 0, 0, 0);
    }

    // ReLU as packed fp16 max after the rounding (as in MlpF16); hidden tiles
    // that are not computed enter as zeros
    __device__ __forceinline__ v4f layer2(const v4f acc[4]) const {
        v4f u = {0.f, 0.f, 0.f, 0.f};
        const v8h zero = {};
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            v8f x;
#pragma unroll
            for (int s = 0; s < 8; ++s) x[s] = 2 * p + s / 4 < NT ? acc[2 * p + s / 4][s % 4] : 0.f;
            const v8h h = __builtin_elementwise_max(__builtin_convertvector(x, v8h), zero);
            u = __builtin_amdgcn_mfma_f32_16x16x32_f16(w2l[p], h, u, 0, 0, 0);
            u = __builtin_amdgcn_mfma_f32_16x16x32_f16(w2h[p], h, u, 0, 0, 0);
        }
        return u;
    }
};
using MlpF16S = MlpF16SM<kC, kH>;

// The MLP policy of fp32 states when none is asked for.
using MlpF32State = MlpF16S;

// Fire bits.  One Philox4x64-10 evaluation gives the draws of a block of 8
// consecutive cells, so a wave evaluates one block per lane and spreads the
// bits with eight ballots (ballot b holds the bit of cell b of each lane's
// block).  Lanes are assigned to row slots of `opr` blocks each: bit
// (slot * opr + o) of ballot b is the bit of cell 8 * (b0(slot) + o) + b,
// where b0(slot) = (canonical index of the slot's first cell) >> 3.
// When rows start on an 8-cell boundary (w % 8 == 0) a 32-cell tile row is
// exactly 4 blocks (opr = 4) and a lane's cells always take the same ballot
// (cell n of a 16-cell group has b = n % 8), so each lane selects its ballot
// once per evaluation; otherwise a row uses opr = 8 and the ballot is
// selected per cell.  The 2D step selects in registers (FireBits below); the
// 3D steps keep the 8 ballots in a small per-wave LDS array and read ballot
// (idx & 7) by address, because there the register select was lowered to a
// private array whose loads the stores then had to wait for.
struct FireBallots {
    uint64_t w[8];
};

__device__ __forceinline__ FireBallots fire_ballots(uint64_t block, uint32_t step, uint32_t level,
                                                    uint32_t batch, uint64_t seed,
                                                    uint64_t threshold) {
    const Philox4x64Out r = philox4x64_10(block, step, level, batch, seed, 0);
    FireBallots f;
#pragma unroll
    for (int b = 0; b < 8; ++b) f.w[b] = __ballot((uint64_t)draw_of(r, (uint32_t)b) < threshold);
    return f;
}

// Ballot b of the set, selected without branches.
__device__ __forceinline__ uint64_t select_ballot(const FireBallots &f, uint32_t b) {
    const uint64_t w01 = (b & 1u) ? f.w[1] : f.w[0];
    const uint64_t w23 = (b & 1u) ? f.w[3] : f.w[2];
    const uint64_t w45 = (b & 1u) ? f.w[5] : f.w[4];
    const uint64_t w67 = (b & 1u) ? f.w[7] : f.w[6];
    const uint64_t w03 = (b & 2u) ? w23 : w01;
    const uint64_t w47 = (b & 2u) ? w67 : w45;
    return (b & 4u) ? w47 : w03;
}

// Plane stride rounded up to 16 words (256 B): measured on gfx950, strides of
// 2, 4 and 12 words mod 16 left the 16-lane plane reads with ~20x more LDS
// bank-conflict cycles than this choice.
constexpr int plane_stride(int cells) { return (cells + 15) / 16 * 16; }
// Workgroups go to the eight XCDs in turn (blockIdx % 8) and each XCD has an
// L2 of its own.  The grid-stride loops of the 3D step kernels map their index
// u to a work item such that the workgroups of one XCD that run at the same
// time take consecutive items (neighbouring tiles of one z run), which then
// find each other's halo rows and columns in that L2 instead of fetching the
// same lines again (measured: 1% off the video step; the 2D row kernel, where
// it measured 2% slower, keeps the plain order).  A bijection of
// [0, rounds * grid) when grid % 8 == 0, the identity otherwise.
constexpr int kXcds = 8;
__device__ __forceinline__ int64_t xcd_item(int64_t u, int grid) {
    if (grid % kXcds) return u;
    const int64_t r = u / grid;
    const int b = (int)(u - r * grid);
    return (r * kXcds + b % kXcds) * (grid / kXcds) + b / kXcds;
}

// Buffer resources: every global access of the step kernel goes through a
// raw buffer descriptor whose range covers only the rows a tile may touch;
// an out-of-range offset (0xffffffff is used for cells outside the grid)
// reads 0 and drops a store.  So no load or store sits behind a branch, the
// compiler sees a fixed sequence of vector-memory operations per tile, and
// waits for the prefetched loads without draining the stores (loads and
// stores share one completion counter).
typedef __amdgpu_buffer_rsrc_t Rsrc;
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
constexpr uint32_t kOut = 0xffffffffu;      // offset that is always out of range
constexpr int kRsrcWord3 = 0x00020000;      // raw buffer, 32-bit data format

__device__ __forceinline__ Rsrc make_rsrc(const void *base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, bytes, kRsrcWord3);
}

// The chunks in which a cell of C channels moves between memory and LDS: 16
// bytes (4 fp32 or 8 fp16 channels), or 8 bytes where a cell is no multiple of
// 16 (fp16, C = 12).  N chunks cover 16 channels, of which the cell fills
// kUsed; the loads of the others take the out-of-range offset and read as zero.
template <typename T, int C> struct CellChunk {
    static constexpr int kBytes = C * (int)sizeof(T) % 16 == 0 ? 16 : 8;
    static constexpr int N = kC * (int)sizeof(T) / kBytes;
    static constexpr int kUsed = C * (int)sizeof(T) / kBytes;
    static_assert(C * (int)sizeof(T) % kBytes == 0 && kUsed <= N, "whole chunks");
    __device__ static __forceinline__ uint4 load(Rsrc r, uint32_t off) {
        if constexpr (kBytes == 16) {
            const v4u x = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
            return make_uint4(x[0], x[1], x[2], x[3]);
        } else {
            const v2u x = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
            return make_uint4(x[0], x[1], 0u, 0u);
        }
    }
    // Chunk q of a cell into LDS channel-quad planes of fp32 (16-byte words,
    // `stride` apart).
    __device__ static __forceinline__ void put(float4 *planes, int stride, int q, int slot,
                                               const uint4 &c) {
        if constexpr (sizeof(T) == 4) {
            planes[q * stride + slot] = make_float4(__uint_as_float(c.x), __uint_as_float(c.y),
                                                    __uint_as_float(c.z), __uint_as_float(c.w));
        } else if constexpr (kBytes == 8) {
            float f[4];
            Storage<__half>::unpack_pair(c.x, f[0], f[1]);
            Storage<__half>::unpack_pair(c.y, f[2], f[3]);
            planes[q * stride + slot] = make_float4(f[0], f[1], f[2], f[3]);
        } else {
            float f[8];
            Storage<__half>::unpack(c, f);
            planes[(2 * q) * stride + slot] = make_float4(f[0], f[1], f[2], f[3]);
            planes[(2 * q + 1) * stride + slot] = make_float4(f[4], f[5], f[6], f[7]);
        }
    }
};

// Residual update of a channel: m is 1 for a cell that fires and 0 for one that
// does not.  The fma returns the state of a cell that does not fire for finite
// u only (and +0 for a state of -0); with kSelectGate it is kept bit for bit
// for any u.
template <class Mlp>
__device__ __forceinline__ float gated(float m, float u, float f) {
    if constexpr (Mlp::kSelectGate)
        return m != 0.f ? f + u : f;
    else
        return fmaf(m, u, f);
}

// Residual update and store of the lane's 4 channels (fp32 values, stored in
// the storage type) through the tile's store descriptor; `off` is the byte
// offset of the cell in it, or kOut for a cell outside the grid.  u is +0 for
// the input channels (zero W2 rows; u finite).
__device__ __forceinline__ void store_quad(float *, Rsrc w, uint32_t off, int g, const v4f &v) {
    const v4u x = {__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]),
                   __float_as_uint(v[3])};
    __builtin_amdgcn_raw_buffer_store_b128(x, w, off == kOut ? kOut : off + 16u * g, 0, 0);
}
__device__ __forceinline__ void store_quad(__half *, Rsrc w, uint32_t off, int g, const v4f &v) {
    const v2u x = {Storage<__half>::pack_pair(v[0], v[1]), Storage<__half>::pack_pair(v[2], v[3])};
    __builtin_amdgcn_raw_buffer_store_b64(x, w, off == kOut ? kOut : off + 8u * g, 0, 0);
}

template <class Mlp, typename T>
__device__ __forceinline__ void update_store(T *tag, Rsrc w, uint32_t off, int g, const float f[8],
                                             const v4f &u, float m) {   // m: 1 fires, 0 keeps
    v4f out;
    out[0] = gated<Mlp>(m, u[0], f[0]);
    out[1] = gated<Mlp>(m, u[1], f[1]);
    out[2] = gated<Mlp>(m, u[2], f[2]);
    out[3] = gated<Mlp>(m, u[3], f[3]);
    store_quad(tag, w, off, g, out);
}

}  // namespace

}  // namespace octnca
