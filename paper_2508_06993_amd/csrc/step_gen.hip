// Fused NCA step on the matrix cores for any model size C / H with C a
// multiple of 4 (Sec. 3.1; supplement S3, Listing 1).  It serves the other
// sizes of the paper's ablation (supplement S10): C / H = 20 / 100, and of 12 /
// 48 the 2D tile layout and what else the specialised kernels of C = 16, H = 64
// do not take.
//
// Layout (generalising the 16 / 64 kernels' lane mapping):
//   lane l of a wave -> cell n = l % 16 of a 16-cell group and lane group
//   g = l / 16.  The 2C features of a cell are taken in K chunks of 32: chunk
//   k holds channel quads q = 4k .. 4k+3, lane group g the quad q = 4k + g as
//   eight K slots (its 4 state channels, then its 4 perception channels).
//   Quads beyond C / 4 are zero slots.  So a lane forms the perception of the
//   channels it owns, and
//   * layer 1, H[j][n] = b1[j] + sum_k W1[j][k] F[k][n], is
//     v_mfma_f32_16x16x32_f16 with A = a 16-unit tile of W1's rows (columns
//     gathered in the slot order above) and B = the lane's 8 features; its
//     accumulator leaves hidden unit 16t + 4g + i of cell n in register i;
//   * two hidden tiles (2p, 2p+1) together are the 8 K slots of lane group g
//     in layer 2's chunk p: slot s <-> hidden unit (2p + s/4) 16 + 4g + s%4,
//     W2's columns gathered to match, so ReLU'd accumulators feed layer 2
//     directly (no hidden activation leaves the registers);
//   * layer 2's output tile k holds channels 16k + 4g + i of cell n, which is
//     the lane's own quad of chunk k: the residual and the store need no
//     exchange.
// A last chunk that holds a single quad (C = 20: quad 4) is not spread over the
// lane groups like that, which would leave three of four lanes idle in its
// perception and three of four K slots and rows empty in its products.  Lane
// group g forms that quad for group g's cells, so one pass serves four groups.
// Its layer-1 operand is brought into two lane groups, against which A holds
// the hi and the lo part of the weights: one product instead of two.  Layer
// 2's rows for it hold hi in lane groups 0 and 1 and lo in 2 and 3: one product
// again, and the two halves are added across the lanes once per four groups.
// (20 / 100, fp32, 1408 x 2048 cells, with the loads below: 132 products and
// 808 vector instructions per 64 cells instead of 192 and 1109, a step 196 ->
// 153 us.)
// Hidden tiles are padded to an even count with zero weights (a tile of padding
// only is left out); W2's rows of
// the input channels (and of channels >= C) are zero, so their update is +0.
// MLP arithmetic: fp32 states take the scaled-fp16 form of the 16 / 64
// kernels (activations times 2^-8 rounded to fp16, weights as fp16 hi + lo,
// two products per weight, fp32 accumulation); fp16 states take fp16
// weights and activations, fp32 accumulation.
//
// Work: a persistent grid loops over tiles of 8 x 32 cells (2D) or
// 2 x 4 x 32 (3D).  A tile and its one-cell halo are staged in LDS as fp32 in
// channel-quad planes (16 consecutive lanes read 16 consecutive 16-byte
// words); the block's weights are converted once into LDS in lane order, and
// each wave reads an MFMA's weight operand once for its four groups.  Fire
// bits: one Philox4x64-10 evaluation per block of 8 consecutive cells of a
// tile row, kept as a byte in LDS.
#include <algorithm>
#include <type_traits>

#include "launch.h"
#include "step_common.h"

namespace octnca {

namespace {

constexpr int kGenThreads = 256;   // 4 waves, 4 groups of 16 cells each
constexpr float kGenScale = 1.f / 256.f;
constexpr int kGenAhead = 6;       // tiles whose fire bits are formed together (240 of 256 lanes, 2D)

template <int C, int H>
struct GenDims {
    static_assert(C % 4 == 0, "channels in whole quads");
    static constexpr int NQ = C / 4;              // channel quads
    static constexpr int NK = (NQ + 3) / 4;       // layer-1 K chunks = layer-2 output tiles
    static constexpr int NT = (H + 15) / 16;      // hidden tiles
    static constexpr int NT2 = (NT + 1) / 2 * 2;  // padded to whole pairs
    static constexpr int NP = NT2 / 2;            // layer-2 K chunks
    static constexpr bool kTail = NK > 1 && NQ % 4 == 1;   // a last chunk of one quad
    static constexpr int NF = kTail ? NK - 1 : NK;         // chunks spread over the lane groups
};

template <int NDIM> struct GenTile;
template <> struct GenTile<2> { static constexpr int TZ = 1, TY = 8, TX = 32; };
template <> struct GenTile<3> { static constexpr int TZ = 2, TY = 4, TX = 32; };

struct WPair {
    v8h hi, lo;
};

// One channel quad through a buffer descriptor (kOut: reads zero, stores
// nothing).
__device__ __forceinline__ float4 load_quad(const float *, Rsrc r, uint32_t off) {
    const v4u x = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
    return make_float4(__uint_as_float(x[0]), __uint_as_float(x[1]), __uint_as_float(x[2]),
                       __uint_as_float(x[3]));
}
__device__ __forceinline__ float4 load_quad(const __half *, Rsrc r, uint32_t off) {
    const v2u v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
    float4 f;
    Storage<__half>::unpack_pair(v[0], f.x, f.y);
    Storage<__half>::unpack_pair(v[1], f.z, f.w);
    return f;
}

// An empty asm that reads and rewrites the value: work before it stays before it.
__device__ __forceinline__ void pin4(float4 &v) {
    asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
}

__device__ __forceinline__ float4 fma4(float4 a, float4 b, float4 c) {
    return make_float4(fmaf(a.x, b.x, c.x), fmaf(a.y, b.y, c.y), fmaf(a.z, b.z, c.z),
                       fmaf(a.w, b.w, c.w));
}

// Feature column of W1 for K slot s of lane group g in chunk k (-1: zero slot).
template <int C>
__device__ __forceinline__ int gen_feature(int k, int g, int s) {
    const int q = 4 * k + g;
    if (q >= C / 4) return -1;
    return s < 4 ? 4 * q + s : C + 4 * q + (s - 4);
}

// Hidden unit of layer 2's K slot s of lane group g in chunk p.
__device__ __forceinline__ int gen_hidden(int p, int g, int s) {
    return (2 * p + s / 4) * 16 + 4 * g + s % 4;
}

// Blocks per CU (4 waves each) that LDS (160 KB per CU) and registers allow:
// 2D C = 12 three (31 KB of LDS each), 2D C = 20 and 3D C = 12 two (66 KB and
// 54 KB), 3D C = 20 one (105 KB).
template <int NDIM, int C>
constexpr int kGenBlocksPerCu = NDIM == 2 ? (C <= 12 ? 3 : 2) : (C <= 12 ? 2 : 1);

template <typename T, int NDIM, int NIN, int C, int H>
__global__ __launch_bounds__(kGenThreads, (kGenBlocksPerCu<NDIM, C>)) void nca_step_gen(
    const T *__restrict__ src, T *__restrict__ dst, int dd, int dh, int dw, int tiles_x,
    int tiles_y, int tiles, const float *__restrict__ conv_w, const float *__restrict__ conv_b,
    const float *__restrict__ w1, const float *__restrict__ b1, const float *__restrict__ w2,
    uint32_t level, uint32_t step, uint32_t batch, uint64_t seed, uint64_t threshold) {
    using D = GenDims<C, H>;
    constexpr bool kSplit = std::is_same_v<T, float>;   // fp32 states: split weights, scaled
    constexpr float kScale = kSplit ? kGenScale : 1.f;
    constexpr int TZ = GenTile<NDIM>::TZ, TY = GenTile<NDIM>::TY, TX = GenTile<NDIM>::TX;
    constexpr int HZ = NDIM == 3 ? TZ + 2 : 1, HY = TY + 2, HX = TX + 2;
    constexpr int NCELL = HZ * HY * HX;
    constexpr int PS = (NCELL + 15) / 16 * 16;          // quad-plane stride (float4s)
    constexpr int TAPS = NDIM == 3 ? 27 : 9;
    constexpr int ROWS = TZ * TY;                        // tile rows of TX cells
    constexpr int BPR = TX / 8 + 1;                      // 8-cell blocks a tile row can touch

    __shared__ float4 halo[D::NQ * PS];
    __shared__ float4 tapw[TAPS][D::NQ];                 // conv weights of quad q, times kScale
    __shared__ float4 cbias[D::NQ];                      // conv bias, times kScale
    __shared__ WPair w1s[D::NT2][D::NF][64];             // layer-1 A operands in lane order
    __shared__ float4 b1s[D::NT2][4];                    // [t][g]: b1[16t + 4g + i] * kScale
    __shared__ WPair w2s[D::NP][D::NF][64];              // layer-2 A operands in lane order
    __shared__ v8h w1t[D::kTail ? D::NT : 1][64];        // the same of a single last quad
    __shared__ v8h w2t[D::kTail ? D::NP : 1][64];
    __shared__ uint32_t fire_bytes[kGenAhead][ROWS][BPR];   // 8 fire bits per block (low byte)

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int n = lane & 15;
    const int g = lane >> 4;

    // ---- weights into LDS (once per block) ----
    for (int i = tid; i < TAPS * D::NQ; i += kGenThreads) {
        const int t = i / D::NQ, q = i % D::NQ;
        tapw[t][q] = make_float4(kScale * conv_w[(4 * q + 0) * TAPS + t],
                                 kScale * conv_w[(4 * q + 1) * TAPS + t],
                                 kScale * conv_w[(4 * q + 2) * TAPS + t],
                                 kScale * conv_w[(4 * q + 3) * TAPS + t]);
    }
    for (int q = tid; q < D::NQ; q += kGenThreads)
        cbias[q] = make_float4(kScale * conv_b[4 * q + 0], kScale * conv_b[4 * q + 1],
                               kScale * conv_b[4 * q + 2], kScale * conv_b[4 * q + 3]);
    for (int i = tid; i < D::NT2 * D::NF * 64; i += kGenThreads) {
        const int l = i % 64, k = (i / 64) % D::NF, t = i / (64 * D::NF);
        const int row = 16 * t + (l & 15), lg = l >> 4;
        v8f x;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int f = gen_feature<C>(k, lg, s);
            // load a valid element for every slot, then zero the padding (a
            // load behind the condition costs a branch and a memory wait)
            const float v = w1[min(row, H - 1) * 2 * C + max(f, 0)];
            x[s] = (row < H && f >= 0) ? v : 0.f;
        }
        WPair wp;
        wp.hi = __builtin_convertvector(x, v8h);
        wp.lo = __builtin_convertvector(x - __builtin_convertvector(wp.hi, v8f), v8h);
        w1s[t][k][l] = wp;
    }
    for (int i = tid; i < D::NT2 * 4; i += kGenThreads) {
        const int t = i / 4, lg = i % 4;
        float b[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int j = 16 * t + 4 * lg + r;
            const float v = b1[min(j, H - 1)];
            b[r] = j < H ? kScale * v : 0.f;
        }
        b1s[t][lg] = make_float4(b[0], b[1], b[2], b[3]);
    }
    for (int i = tid; i < D::NP * D::NF * 64; i += kGenThreads) {
        const int l = i % 64, k = (i / 64) % D::NF, p = i / (64 * D::NF);
        const int ch = 16 * k + (l & 15), lg = l >> 4;
        v8f x;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int j = gen_hidden(p, lg, s);
            const float v = w2[min(ch, C - 1) * H + min(j, H - 1)];
            x[s] = (ch >= NIN && ch < C && j < H) ? v * (1.f / kScale) : 0.f;
        }
        WPair wp;
        wp.hi = __builtin_convertvector(x, v8h);
        wp.lo = __builtin_convertvector(x - __builtin_convertvector(wp.hi, v8f), v8h);
        w2s[p][k][l] = wp;
    }

    if constexpr (D::kTail) {
        // lane groups 2 and 3 hold the lo part of split weights
        auto part = [&](const v8f &x, int lg) {
            const v8h hi = __builtin_convertvector(x, v8h);
            const v8h lo = __builtin_convertvector(x - __builtin_convertvector(hi, v8f), v8h);
            return kSplit && lg >= 2 ? lo : hi;
        };
        for (int i = tid; i < D::NT * 64; i += kGenThreads) {
            const int l = i % 64, t = i / 64, row = 16 * t + (l & 15);
            v8f x;
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const float v = w1[min(row, H - 1) * 2 * C + gen_feature<C>(D::NF, 0, s)];
                x[s] = row < H ? v : 0.f;
            }
            w1t[t][l] = part(x, l >> 4);
        }
        for (int i = tid; i < D::NP * 64; i += kGenThreads) {
            const int l = i % 64, p = i / 64;
            const int ch = 16 * D::NF + (l & 3);   // rows 4 r + i: channel i of the quad
            v8f x;
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int j = gen_hidden(p, l >> 4, s);
                const float v = w2[ch * H + min(j, H - 1)];
                x[s] = j < H ? v * (1.f / kScale) : 0.f;
            }
            w2t[p][l] = part(x, (l & 15) >> 2);
        }
    }

    // LDS index of group grp's cell (relative to a quad plane), and its
    // position in the tile: 2D rows 2 wave + grp / 2; 3D plane wave / 2,
    // rows 2 (wave % 2) + grp / 2; columns 16 (grp % 2) + n.
    int lz[4], ly[4], lx[4], centre[4];
#pragma unroll
    for (int grp = 0; grp < 4; ++grp) {
        lz[grp] = NDIM == 3 ? wave / 2 : 0;
        ly[grp] = NDIM == 3 ? 2 * (wave % 2) + grp / 2 : 2 * wave + grp / 2;
        lx[grp] = 16 * (grp % 2) + n;
        centre[grp] = ((NDIM == 3 ? lz[grp] + 1 : 0) * HY + ly[grp] + 1) * HX + lx[grp] + 1;
    }

    // the cell of the lane's own group (group g), for a single last quad
    const int own_centre = ((NDIM == 3 ? wave / 2 + 1 : 0) * HY +
                            (NDIM == 3 ? 2 * (wave % 2) : 2 * wave) + g / 2 + 1) * HX +
                           16 * (g % 2) + n + 1;

    // The next tile's halo quads are loaded into registers while the current
    // tile is computed and written to LDS after it, so the loads' latency
    // overlaps the compute.  Thread t takes quad t % NQ of cells t / NQ + CPT j
    // (j = 0, 1, ..), whose halo coordinates follow from the first by additions
    // and whose LDS words lie a constant apart; offsets are 32 bits from the
    // halo's first cell.  (Deriving cell, row and column anew by division took
    // about 400 of 990 vector instructions per 64 cells.)
    constexpr int CPT = kGenThreads / D::NQ;             // cells per turn of the block
    constexpr int LPT = (NCELL + CPT - 1) / CPT;
    constexpr uint32_t kCell = C * (uint32_t)sizeof(T);
    const int my_q = tid % D::NQ, my_cell = tid < CPT * D::NQ ? tid / D::NQ : NCELL;
    const int my_x = my_cell % HX, my_y = my_cell / HX % HY, my_z = my_cell / (HX * HY);
    const uint32_t row_cells = (uint32_t)dw, plane_cells = (uint32_t)dh * (uint32_t)dw;
    float4 pre[LPT];
    auto issue = [&](int tile) {
        const int x0 = (tile % tiles_x) * TX, y0 = ((tile / tiles_x) % tiles_y) * TY;
        const int z0 = (tile / (tiles_x * tiles_y)) * TZ;
        // the halo's first cell (it may lie outside the grid: its lanes do not load)
        const int64_t first =
            ((int64_t)(NDIM == 3 ? z0 - 1 : z0) * dh + (y0 - 1)) * dw + (x0 - 1);
        const Rsrc r = make_rsrc(src + first * C, tile < tiles ? kOut - 1 : 0u);
        int hx = my_x, hy = my_y, hz = my_z;
#pragma unroll
        for (int j = 0; j < LPT; ++j) {
            const bool ok = my_cell + j * CPT < NCELL && (uint32_t)(x0 - 1 + hx) < (uint32_t)dw &&
                            (uint32_t)(y0 - 1 + hy) < (uint32_t)dh &&
                            (NDIM == 2 || (uint32_t)(z0 - 1 + hz) < (uint32_t)dd);
            uint32_t cell = (uint32_t)hy * row_cells + (uint32_t)hx;
            if constexpr (NDIM == 3) cell += (uint32_t)hz * plane_cells;
            pre[j] = load_quad(src, r, ok ? cell * kCell + my_q * (uint32_t)(4 * sizeof(T)) : kOut);
            hx += CPT % HX;
            hy += CPT / HX;
            if (hx >= HX) {
                hx -= HX;
                ++hy;
            }
            if (NDIM == 3 && hy >= HY) {
                hy -= HY;
                ++hz;
            }
        }
    };
    issue(blockIdx.x);

    int ahead = 0;   // tile's place among those the fire bits are kept for
    for (int tile = blockIdx.x; tile < tiles;
         tile += gridDim.x, ahead = ahead + 1 < kGenAhead ? ahead + 1 : 0) {
        const int tx = tile % tiles_x;
        const int ty = (tile / tiles_x) % tiles_y;
        const int tz = tile / (tiles_x * tiles_y);
        const int x0 = tx * TX, y0 = ty * TY, z0 = tz * TZ;

        __syncthreads();   // weights written / the previous tile's readers are done
        // ---- halo tile: fp32 channel-quad planes, zero outside the grid ----
#pragma unroll
        for (int j = 0; j < LPT; ++j)
            if (my_cell + j * CPT < NCELL) halo[my_q * PS + my_cell + j * CPT] = pre[j];
        // ---- fire bits: block b0(row) + k of each tile row, for this block's
        // next kGenAhead tiles at once (a tile has too few rows for all lanes) ----
        if (ahead == 0) {
            for (int i = tid; i < kGenAhead * ROWS * BPR; i += kGenThreads) {
                const int a = i / (ROWS * BPR), r = i / BPR % ROWS, k = i % BPR;
                const int t2 = min(tile + a * (int)gridDim.x, tiles - 1);
                const int z = t2 / (tiles_x * tiles_y) * TZ + r / TY;
                const int y = (t2 / tiles_x) % tiles_y * TY + r % TY;
                const uint64_t idx0 = ((uint64_t)z * dh + y) * dw + t2 % tiles_x * TX;
                const Philox4x64Out o =
                    philox4x64_10((idx0 >> 3) + k, step, level, batch, seed, 0);
                uint32_t byte = 0;
#pragma unroll
                for (int b = 0; b < 8; ++b) byte |= ((uint64_t)draw_of(o, b) < threshold ? 1u : 0u) << b;
                fire_bytes[a][r][k] = byte;
            }
        }
        __syncthreads();
        issue(tile + gridDim.x);   // the next tile's loads, in flight during the compute

        // ---- features: chunk k of group grp = quad 4k + g of its cell; a
        // tap's weights are read once and applied to the four groups ----
        v8h fe[4][D::NF];
        float4 st[4][D::NF];   // the lane's state quads (for the residual)
#pragma unroll
        for (int k = 0; k < D::NF; ++k) {
            const int q = 4 * k + g;
            const bool qv = q < D::NQ;
            const int qc = qv ? q : D::NQ - 1;
            const float4 *pl = halo + qc * PS;
            float4 p[4];
            const float4 cb = cbias[qc];
#pragma unroll
            for (int grp = 0; grp < 4; ++grp) p[grp] = cb;
#pragma unroll
            for (int t = 0; t < TAPS; ++t) {
                const int dz = NDIM == 3 ? t / 9 - 1 : 0;
                const int dy = (t / 3) % 3 - 1, dx = t % 3 - 1;
                const float4 w = tapw[t][qc];
#pragma unroll
                for (int grp = 0; grp < 4; ++grp)
                    p[grp] = fma4(w, pl[centre[grp] + (dz * HY + dy) * HX + dx], p[grp]);
                // keep the compiler from hoisting every tap's reads at once
#pragma unroll
                for (int grp = 0; grp < 4; ++grp) pin4(p[grp]);
            }
#pragma unroll
            for (int grp = 0; grp < 4; ++grp) {
                const float4 sv = pl[centre[grp]];
                st[grp][k] = sv;
                v8f x = {sv.x * kScale, sv.y * kScale, sv.z * kScale, sv.w * kScale,
                         p[grp].x, p[grp].y, p[grp].z, p[grp].w};
                if (!qv) x = v8f{};
                fe[grp][k] = __builtin_convertvector(x, v8h);
            }
        }

        // the single last quad of group g's cell, and for each group its layer-1
        // operand: in lane groups grp % 2 and grp % 2 + 2 (split weights: hi and
        // lo), or in lane group grp; zero in the others
        float4 st_t = make_float4(0.f, 0.f, 0.f, 0.f);
        v8h fe_t[D::kTail ? 4 : 1];
        if constexpr (D::kTail) {
            const float4 *pl = halo + (D::NQ - 1) * PS + own_centre;
            float4 p = cbias[D::NQ - 1];
#pragma unroll
            for (int t = 0; t < TAPS; ++t) {
                const int dz = NDIM == 3 ? t / 9 - 1 : 0;
                const int dy = (t / 3) % 3 - 1, dx = t % 3 - 1;
                p = fma4(tapw[t][D::NQ - 1], pl[(dz * HY + dy) * HX + dx], p);
            }
            st_t = pl[0];
            const v8f x = {st_t.x * kScale, st_t.y * kScale, st_t.z * kScale, st_t.w * kScale,
                           p.x, p.y, p.z, p.w};
            const v4u w = __builtin_bit_cast(v4u, __builtin_convertvector(x, v8h));
            v4u f[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if constexpr (kSplit) {
                    const auto h = __builtin_amdgcn_permlane32_swap(w[i], w[i], false, false);
                    const bool even = (g & 1) == 0;   // h[0]: lanes 0 .. 31 in both halves
                    f[0][i] = even ? h[0] : 0u;
                    f[1][i] = even ? 0u : h[0];
                    f[2][i] = even ? h[1] : 0u;
                    f[3][i] = even ? 0u : h[1];
                } else {
#pragma unroll
                    for (int grp = 0; grp < 4; ++grp) f[grp][i] = g == grp ? w[i] : 0u;
                }
            }
#pragma unroll
            for (int grp = 0; grp < 4; ++grp) fe_t[grp] = __builtin_bit_cast(v8h, f[grp]);
        }

        // ---- MLP: per hidden-tile pair, layer 1 then its share of layer 2 ----
        v4f u[4][D::NF], u_t[D::kTail ? 4 : 1];
#pragma unroll
        for (int grp = 0; grp < 4; ++grp) {
#pragma unroll
            for (int k = 0; k < D::NF; ++k) u[grp][k] = v4f{0.f, 0.f, 0.f, 0.f};
            if constexpr (D::kTail) u_t[grp] = v4f{0.f, 0.f, 0.f, 0.f};
        }
        const v8h zero = {};
#pragma unroll
        for (int pr = 0; pr < D::NP; ++pr) {
            v4f acc[4][2];
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2) {
                const int t = 2 * pr + h2;
                if (t >= D::NT) continue;   // padding only
                const float4 bb = b1s[t][g];
#pragma unroll
                for (int grp = 0; grp < 4; ++grp) acc[grp][h2] = v4f{bb.x, bb.y, bb.z, bb.w};
#pragma unroll
                for (int k = 0; k < D::NF; ++k) {
                    const WPair w = w1s[t][k][lane];
#pragma unroll
                    for (int grp = 0; grp < 4; ++grp) {
                        if constexpr (kSplit)
                            acc[grp][h2] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                                w.lo, fe[grp][k], acc[grp][h2], 0, 0, 0);
                        acc[grp][h2] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                            w.hi, fe[grp][k], acc[grp][h2], 0, 0, 0);
                    }
                }
                if constexpr (D::kTail) {
                    const v8h w = w1t[t][lane];
#pragma unroll
                    for (int grp = 0; grp < 4; ++grp)
                        acc[grp][h2] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                            w, fe_t[grp], acc[grp][h2], 0, 0, 0);
                }
            }
            v8h hh[4];
#pragma unroll
            for (int grp = 0; grp < 4; ++grp) {
                v8f x;
#pragma unroll
                for (int s = 0; s < 8; ++s)
                    x[s] = 2 * pr + s / 4 < D::NT ? acc[grp][s / 4][s % 4] : 0.f;
                // ReLU after the rounding to fp16 (monotonic, keeps zero)
                hh[grp] = __builtin_elementwise_max(__builtin_convertvector(x, v8h), zero);
            }
#pragma unroll
            for (int k = 0; k < D::NF; ++k) {
                const WPair w = w2s[pr][k][lane];
#pragma unroll
                for (int grp = 0; grp < 4; ++grp) {
                    if constexpr (kSplit)
                        u[grp][k] =
                            __builtin_amdgcn_mfma_f32_16x16x32_f16(w.lo, hh[grp], u[grp][k], 0, 0, 0);
                    u[grp][k] =
                        __builtin_amdgcn_mfma_f32_16x16x32_f16(w.hi, hh[grp], u[grp][k], 0, 0, 0);
                }
            }
            if constexpr (D::kTail) {
                const v8h w = w2t[pr][lane];
#pragma unroll
                for (int grp = 0; grp < 4; ++grp)
                    u_t[grp] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w, hh[grp], u_t[grp], 0, 0, 0);
            }
        }

        // ---- fire gate, residual, store (out of place) ----
        const int64_t first = ((int64_t)z0 * dh + y0) * dw + x0;
        const Rsrc wr = make_rsrc(dst + first * C, kOut - 1);
        // offset and fire bit of the cell at row ly (plane lz) and column lx of the tile
        auto cell_off = [&](int lz_, int ly_, int lx_) -> uint32_t {
            const uint32_t cell =
                (NDIM == 3 ? (uint32_t)lz_ * plane_cells : 0u) + (uint32_t)ly_ * row_cells + (uint32_t)lx_;
            return z0 + lz_ < dd && y0 + ly_ < dh && x0 + lx_ < dw ? cell * kCell : kOut;
        };
        auto cell_fires_at = [&](int lz_, int ly_, int lx_) -> bool {
            // the row's first cell is bit idx0 % 8 of its first byte
            const uint32_t idx0 = ((uint32_t)(z0 + lz_) * (uint32_t)dh + (uint32_t)(y0 + ly_)) * row_cells +
                                  (uint32_t)x0;
            const uint32_t bit = (idx0 & 7u) + (uint32_t)lx_;
            return (fire_bytes[ahead][lz_ * TY + ly_][bit >> 3] >> (bit & 7u)) & 1u;
        };
        auto put = [&](uint32_t off, int q, bool fires, const float4 &s, const v4f &du) {
            const v4f o = {fires ? s.x + du[0] : s.x, fires ? s.y + du[1] : s.y,
                           fires ? s.z + du[2] : s.z, fires ? s.w + du[3] : s.w};
            store_quad(dst, wr, off, q, o);
        };
#pragma unroll
        for (int grp = 0; grp < 4; ++grp) {
            const uint32_t off = cell_off(lz[grp], ly[grp], lx[grp]);
            const bool fires = cell_fires_at(lz[grp], ly[grp], lx[grp]);
#pragma unroll
            for (int k = 0; k < D::NF; ++k) {
                const int q = 4 * k + g;
                put(q < D::NQ ? off : kOut, q, fires, st[grp][k], u[grp][k]);
            }
        }
        if constexpr (D::kTail) {
            // lane group g: its group's update (split: the hi part from lane
            // group g's rows, the lo part from the other half's, or the reverse)
            float du[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                du[i] = g == 0 ? u_t[0][i] : g == 1 ? u_t[1][i] : g == 2 ? u_t[2][i] : u_t[3][i];
                if constexpr (kSplit) {
                    const float y = g == 2   ? u_t[0][i]
                                    : g == 3 ? u_t[1][i]
                                    : g == 0 ? u_t[2][i]
                                             : u_t[3][i];
                    const auto h = __builtin_amdgcn_permlane32_swap(
                        __float_as_uint(y), __float_as_uint(y), false, false);
                    du[i] += __uint_as_float(lane < 32 ? h[1] : h[0]);
                }
            }
            const int tz_ = NDIM == 3 ? wave / 2 : 0;
            const int ty_ = (NDIM == 3 ? 2 * (wave % 2) : 2 * wave) + g / 2, tx_ = 16 * (g % 2) + n;
            put(cell_off(tz_, ty_, tx_), 4 * D::NF, cell_fires_at(tz_, ty_, tx_), st_t,
                v4f{du[0], du[1], du[2], du[3]});
        }
    }
}

template <typename T, int NDIM, int NIN, int C, int H>
hipError_t launch_gen_t(const StepArgs &a, const void *src, void *dst, hipStream_t stream) {
    constexpr int TZ = GenTile<NDIM>::TZ, TY = GenTile<NDIM>::TY, TX = GenTile<NDIM>::TX;
    const int64_t tiles_x = (a.ext.w + TX - 1) / TX;
    const int64_t tiles_y = (a.ext.h + TY - 1) / TY;
    const int64_t tiles_z = (a.ext.d + TZ - 1) / TZ;
    const int64_t tiles = tiles_x * tiles_y * tiles_z;
    if (tiles == 0) return hipSuccess;
    // 32-bit offsets within a tile's halo planes and rows; larger ones go to
    // the vector kernel
    const int64_t span = ((NDIM == 3 ? (TZ + 2) * a.ext.h : 0) + TY + 2) * a.ext.w;
    if (span >= (int64_t(1) << 32) / (C * (int64_t)sizeof(T)) - 64)
        return launch_step_valu(a, src, dst, stream);
    if (tiles > INT32_MAX || tiles_x * tiles_y > INT32_MAX) return hipErrorInvalidValue;
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess)
        (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    const int grid =
        (int)std::min<int64_t>(tiles, (int64_t)std::max(cus, 1) * kGenBlocksPerCu<NDIM, C>);
    nca_step_gen<T, NDIM, NIN, C, H><<<grid, kGenThreads, 0, stream>>>(
        (const T *)src, (T *)dst, (int)a.ext.d, (int)a.ext.h, (int)a.ext.w, (int)tiles_x,
        (int)tiles_y, (int)tiles, a.w.conv_w, a.w.conv_b, a.w.w1, a.w.b1, a.w.w2, a.level, a.step,
        a.batch, a.seed, a.threshold);
    return hipGetLastError();
}

template <typename T, int C, int H>
hipError_t launch_gen_size(const StepArgs &a, const void *src, void *dst, hipStream_t stream) {
    if (a.ndim == 2) {
        if (a.n_in == 1) return launch_gen_t<T, 2, 1, C, H>(a, src, dst, stream);
        if (a.n_in == 3) return launch_gen_t<T, 2, 3, C, H>(a, src, dst, stream);
    } else if (a.ndim == 3) {
        if (a.n_in == 1) return launch_gen_t<T, 3, 1, C, H>(a, src, dst, stream);
        if (a.n_in == 3) return launch_gen_t<T, 3, 3, C, H>(a, src, dst, stream);
    }
    return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_gen_dtype(const StepArgs &a, const void *src, void *dst, hipStream_t stream) {
    if (a.channels == 12 && a.hidden == 48) return launch_gen_size<T, 12, 48>(a, src, dst, stream);
    if (a.channels == 20 && a.hidden == 100) return launch_gen_size<T, 20, 100>(a, src, dst, stream);
    return hipErrorInvalidValue;
}

}  // namespace

bool step_gen_serves(const StepArgs &a) {
    return (a.channels == 12 && a.hidden == 48) || (a.channels == 20 && a.hidden == 100);
}

hipError_t launch_step_gen(const StepArgs &a, const void *src, void *dst, hipStream_t stream) {
    if (!step_gen_serves(a)) return hipErrorInvalidValue;
    return a.dtype == Dtype::F32 ? launch_gen_dtype<float>(a, src, dst, stream)
                                 : launch_gen_dtype<__half>(a, src, dst, stream);
}

}  // namespace octnca
