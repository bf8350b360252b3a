// Backward of the NCA step on large tiles, for C = 16, H = 64 (fp32 states):
// several steps of a 2D level, or one step of a 3D level, per launch.
//
// The per-step quantities are those of train.hip: for a cell with state S and
// G' = dL/dS' the activations are recomputed (a = W1 f + b1, h = relu(a)),
//   gu = m G' (hidden channels), ga = (W2^T gu) [a > 0], [gS, gP] = W1^T ga,
//   G = G' + gS + conv^T(gP), and the weight gradients are sums over cells of
//   ga f^T, gu h^T, ga, gP and gP S(neighbour).
//
// A block of 8 waves owns a tile.  Its states come from the tape, one step at
// a time (the next one is loaded while the current one is computed); G' and gP
// stay in LDS between the steps of a launch.  Step s of k runs on the tile
// grown by k - 1 - s cells on each side (conv^T takes one cell of halo per
// step), but only the tile's own cells enter the weight gradients, which
// accumulate in registers over all cells and steps and are written once per
// launch, as one row per block.  Before, a launch ran one step on 64-cell
// blocks: it gathered the weights from memory in every wave and read and wrote
// a row of 3.4 K partial sums per 64 cells (52.6 us for a step of 320^2 cells
// where its MFMAs take 12 us; 11 us for a step of 20^2 to 80^2 cells).
//
// All contractions are fp32 products with fp32 sums (v_mfma_f32_16x16x4_f32)
// in the lane layout of bwd_cell_mfma: lane (n, g) holds channel quad g of
// cell n, every product but the outer ones of the weight gradients takes the
// lane's own values as its operand, and those go through a private LDS patch
// of the wave (16 cells at a time).
#include <algorithm>
#include <type_traits>

#include "launch.h"
#include "step_common.h"

namespace octnca {

namespace {

constexpr int kBwWaves = 8;
constexpr int kBwThreads = 64 * kBwWaves;
constexpr int kBwMaxSteps = 8;
constexpr int kBwRegion = 24;                 // 2D: tile + 2 k at most (LDS row stride)
constexpr int kBwRegion3 = 6 * 10 * 10;       // 3D: 4 x 8 x 8 tile with its halo
constexpr int kPatch = 84;                    // floats per cell of a wave's patch

// Weight-gradient entries of a row: dW1 (H x 2C), dW2 (C x H), db1, dconv_b,
// dconv_w (C x taps).
template <int TAPS> struct BwRow {
    static constexpr int C = 16, H = 64;
    static constexpr int W1 = 0, W2 = 2 * C * H, B1 = 3 * C * H, CB = B1 + H, CW = CB + C,
                         N = CW + C * TAPS;
};

struct BwArgs {
    const float *states;   // the state before step `step`; the one before step - s lies s states
                           // of the level before it
    const float *gout;     // G' of step `step`, or its part without conv^T(gp_prev)
    const float *gp_prev;  // [cells][C] perception gradient of step + 1, or null
    float *gpart, *gp;     // G' + gS and gP of the launch's last (lowest) step, [cells][C]
    float *partial;        // one row per block
    const float *conv_w, *conv_b, *w1, *b1, *w2;
    uint64_t seed, threshold;
    int dd, dh, dw;
    int tile, tiles, tiles_x, tiles_y, steps, accumulate;
    uint32_t level, step, batch;   // step: the first (highest) one
};

template <int NDIM, int NIN>
__global__ __launch_bounds__(kBwThreads, 1) void bwd_block(const BwArgs A) {
    constexpr int C = 16, H = 64;
    constexpr int TAPS = NDIM == 3 ? 27 : 9;
    using G = BwRow<TAPS>;
    constexpr int kCells = NDIM == 3 ? kBwRegion3 : kBwRegion * kBwRegion;   // with halo
    constexpr int kInner = NDIM == 3 ? 256 : (kBwRegion - 2) * (kBwRegion - 2);
    constexpr int kRows = NDIM == 3 ? 32 : kBwRegion - 2;
    constexpr int kLd1 = H + 4, kLd2 = C + 4;
    struct Work {
        float4 s[4][kCells];         // S, channel quads
        float4 gp[4][kCells];        // gP
        float4 g[4][kInner];         // G'
        float w1t[2 * C * kLd1];     // W1^T [feature][hidden]
        float w2t[H * kLd2];         // W2^T [hidden][channel], 0 for input channels
        float b1[H];
        float4 kw[TAPS][4], kb[4];   // conv weights [tap][quad], bias [quad]
        float patch[kBwWaves][16 * kPatch];
        uint64_t fire[kBwMaxSteps][kRows];
    };
    // epilogue: the waves' sums, in the same space
    struct Sums {
        float dw[kBwWaves][3 * C * H];
        float db[kBwWaves][H + C];
        float dk[kBwWaves][C * 9];
    };
    union Shared {
        Work w;
        Sums s;
        __device__ Shared() {}
    };
    __shared__ Shared sh;
    static_assert(sizeof(Shared) <= 160 * 1024, "LDS of a CU");
    Work &L = sh.w;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int k = NDIM == 3 ? 1 : A.steps;
    const int tsx = NDIM == 3 ? 8 : A.tile, tsy = NDIM == 3 ? 8 : A.tile, tsz = NDIM == 3 ? 4 : 1;
    int x0 = 0, y0 = 0, z0 = 0, ry0 = 0, rx0 = 0;   // the current tile
    const int64_t cells = (int64_t)A.dd * A.dh * A.dw;
    // LDS grid: s and gp hold rows of hx cells (3D: planes of 10 x 10), g the
    // same without the outermost ring
    const int hx = NDIM == 3 ? 10 : A.tile + 2 * k;
    const int ncell = NDIM == 3 ? kBwRegion3 : hx * hx;
    auto at = [&](int z, int y, int x) {
        const int p = (y - ry0) * hx + x - rx0;
        return NDIM == 3 ? p + (z - z0 + 1) * 100 : p;
    };
    auto at_g = [&](int z, int y, int x) {
        return NDIM == 3 ? ((z - z0) * 8 + y - y0) * 8 + x - x0
                         : (y - ry0 - 1) * (hx - 2) + x - rx0 - 1;
    };
    // LDS cell i -> grid cell; false outside the grid
    const uint32_t hmagic = (65536u + hx - 1) / hx;   // i / hx, i < 600
    auto grid_of = [&](int i, int &z, int &y, int &x) {
        int r = i;
        z = 0;
        if constexpr (NDIM == 3) {
            const int zz = i / 100;
            z = z0 + zz - 1;
            r = i - zz * 100;
        }
        const int yy = (int)(((uint32_t)r * hmagic) >> 16);
        y = ry0 + yy;
        x = rx0 + r - yy * hx;
        return x >= 0 && x < A.dw && y >= 0 && y < A.dh && z >= 0 && z < A.dd;
    };
    constexpr int kLoads = (4 * kCells + kBwThreads - 1) / kBwThreads;
    // Loads of one [cells][C] array over the LDS grid: word i of the block is
    // quad i / 16 % 4 of cell (i / 64) * 16 + i % 16, so a wave reads whole
    // lines and writes consecutive words of a plane.
    auto load_cells = [&](const float *src, float4 (&v)[kLoads]) {
        const Rsrc r = make_rsrc(src, src ? (uint32_t)(cells * C * 4) : 0u);
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
            const int i = j * kBwThreads + (int)threadIdx.x;
            const int cell = (i >> 6) * 16 + (i & 15), q = (i >> 4) & 3;
            int z, y, x;
            const bool ok = grid_of(cell, z, y, x) && cell < ncell;
            const uint32_t idx = (uint32_t)((z * A.dh + y) * A.dw + x);
            const v4u t = __builtin_amdgcn_raw_buffer_load_b128(
                r, ok ? idx * (C * 4) + q * 16 : kOut, 0, 0);
            v[j] = make_float4(__uint_as_float(t[0]), __uint_as_float(t[1]), __uint_as_float(t[2]),
                               __uint_as_float(t[3]));
        }
    };
    auto put_cells = [&](float4 (&plane)[4][kCells], const float4 (&v)[kLoads]) {
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
            const int i = j * kBwThreads + (int)threadIdx.x;
            const int cell = (i >> 6) * 16 + (i & 15), q = (i >> 4) & 3;
            if (cell < ncell) plane[q][cell] = v[j];
        }
    };
    auto state_of = [&](int s) { return A.states - (int64_t)s * cells * C; };
    // the region of step s: the tile grown by e cells, clipped to the grid
    struct Rect {
        int ya, yb, xa, xb;
    };
    auto region = [&](int e) {
        return Rect{max(0, y0 - e), min(A.dh, y0 + tsy + e), max(0, x0 - e), min(A.dw, x0 + tsx + e)};
    };

    // G' of a region in LDS += the transposed convolution of gp
    auto conv_t = [&](const Rect r) {
        const int w = r.xb - r.xa, h = r.yb - r.ya;
        const int count = NDIM == 3 ? 256 : w * h;
        const uint32_t magic = (65536u + w - 1) / w;
        const int q = lane >> 4;
        for (int i = wave * 16 + (lane & 15); i < (count + 15) / 16 * 16; i += kBwWaves * 16) {
            int z = 0, y, x;
            if constexpr (NDIM == 3) {
                z = z0 + i / 64;
                y = y0 + (i >> 3) % 8;
                x = x0 + i % 8;
            } else {
                const int yy = (int)(((uint32_t)i * magic) >> 16);
                y = r.ya + yy;
                x = r.xa + i - yy * w;
            }
            const bool ok = i < count && x < A.dw && y < A.dh && z < A.dd;
            if (!ok) continue;
            float4 v = L.g[q][at_g(z, y, x)];
            {
                const int p = at(z, y, x);
                // cell p receives K[c][t] gP[p - o_t] from each tap t
#pragma unroll
                for (int t = 0; t < TAPS; ++t) {
                    const int dz = NDIM == 3 ? t / 9 - 1 : 0, dy = (t / 3) % 3 - 1, dx = t % 3 - 1;
                    const float4 a = L.gp[q][p - dz * 100 - dy * hx - dx];
                    const float4 c = L.kw[t][q];
                    v.x = fmaf(c.x, a.x, v.x);
                    v.y = fmaf(c.y, a.y, v.y);
                    v.z = fmaf(c.z, a.z, v.z);
                    v.w = fmaf(c.w, a.w, v.w);
                }
            }
            L.g[q][at_g(z, y, x)] = v;
        }
    };
    // the cells of g among loaded ones (all but the outermost ring)
    auto put_g = [&](const float4 (&v)[kLoads]) {
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
            const int i = j * kBwThreads + (int)threadIdx.x;
            const int cell = (i >> 6) * 16 + (i & 15), q = (i >> 4) & 3;
            int z, y, x;
            const bool in = grid_of(cell, z, y, x) && cell < ncell;
            const bool inner = NDIM == 3 ? z >= z0 && z < z0 + 4 && y >= y0 && y < y0 + 8 &&
                                               x >= x0 && x < x0 + 8
                                         : y > ry0 && y < ry0 + hx - 1 && x > rx0 && x < rx0 + hx - 1;
            if (in && inner) L.g[q][at_g(z, y, x)] = v[j];
        }
    };
    // ---- weights, one copy per block; gathered from LDS ----
    float wv[6], kv[TAPS * C / kBwThreads + 1], rest;
    {
        const int t = threadIdx.x;
#pragma unroll
        for (int j = 0; j < 4; ++j) wv[j] = A.w1[t + j * kBwThreads];
#pragma unroll
        for (int j = 0; j < 2; ++j) wv[4 + j] = A.w2[t + j * kBwThreads];
#pragma unroll
        for (int j = 0; j < TAPS * C / kBwThreads + 1; ++j)
            kv[j] = A.conv_w[min(t + j * kBwThreads, TAPS * C - 1)];
        rest = t < H ? A.b1[t] : A.conv_b[t & 15];
    }
    {
        const int t = threadIdx.x;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = t + j * kBwThreads;
            L.w1t[(i % (2 * C)) * kLd1 + i / (2 * C)] = wv[j];
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int i = t + j * kBwThreads;
            L.w2t[(i % H) * kLd2 + i / H] = i / H < NIN ? 0.f : wv[4 + j];
        }
#pragma unroll
        for (int j = 0; j < TAPS * C / kBwThreads + 1; ++j) {
            const int i = t + j * kBwThreads;
            if (i < TAPS * C)
                reinterpret_cast<float *>(&L.kw[i % TAPS][i / TAPS / 4])[i / TAPS % 4] = kv[j];
        }
        if (t < H) L.b1[t] = rest;
        if (t >= H && t < H + C) reinterpret_cast<float *>(L.kb)[t & 15] = rest;
    }
    __syncthreads();

    // the wave's weight-gradient sums over its cells and the launch's steps
    v4f dw1[4][2], dw2[4];
    float db1[4][4], dcb[4], dcw[NDIM == 2 ? 9 : 1][4];
    auto clear = [&]() {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        dw1[t][0] = dw1[t][1] = dw2[t] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 4; ++i) db1[t][i] = 0.f;
        dcb[t] = 0.f;
    }
#pragma unroll
    for (int t = 0; t < (NDIM == 2 ? 9 : 1); ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) dcw[t][i] = 0.f;
    };
    if constexpr (NDIM == 3) clear();
    constexpr int kShare = 8;   // lanes per dconv_w job (3D)
    float kacc[3][4] = {};
    const int kjob = threadIdx.x / kShare;
    // 3D: the block's tiles in turn, the sums kept (2D: one tile per block; the
    // registers of its larger sums do not last over another tile's loads)
    bool more = true;
    for (int tile = blockIdx.x; more; tile += gridDim.x) {
    more = NDIM == 3 && tile + (int)gridDim.x < A.tiles;
    {
        int bi = tile;
        const int bx = bi % A.tiles_x;
        bi /= A.tiles_x;
        const int by = bi % A.tiles_y;
        x0 = bx * tsx;
        y0 = by * tsy;
        z0 = (bi / A.tiles_y) * tsz;
        ry0 = y0 - (NDIM == 3 ? 1 : k);
        rx0 = x0 - (NDIM == 3 ? 1 : k);
    }
    float4 sv[kLoads], gv[kLoads], ov[kLoads];
    load_cells(state_of(0), sv);
    load_cells(A.gp_prev, gv);           // zeros without one
    load_cells(A.gout, ov);
    __syncthreads();   // the previous tile is done with LDS
    const Rect r0 = region(k - 1);
    {
        // bit (idx0 & 7) + x - xa of a row's word is the draw of cell x
        const int rows = NDIM == 3 ? 32 : r0.yb - r0.ya;
        const int nb = (r0.xb - r0.xa + 14) >> 3;
        for (int i = threadIdx.x; i < k * rows * nb; i += kBwThreads) {
            const int s = i / (rows * nb);
            const int rb = i - s * rows * nb;
            const int row = rb / nb, b = rb - row * nb;
            const int z = NDIM == 3 ? min(z0 + row / 8, A.dd - 1) : 0;
            const int y = NDIM == 3 ? min(y0 + row % 8, A.dh - 1) : r0.ya + row;
            const uint64_t b0 = (((uint64_t)z * A.dh + y) * A.dw + r0.xa) >> 3;
            const Philox4x64Out p =
                philox4x64_10(b0 + b, A.step - s, A.level, A.batch, A.seed, 0);
            uint32_t bits = 0;
#pragma unroll
            for (int c = 0; c < 8; ++c)
                bits |= ((uint64_t)draw_of(p, (uint32_t)c) < A.threshold ? 1u : 0u) << c;
            reinterpret_cast<uint8_t *>(&L.fire[s][row])[b] = (uint8_t)bits;
        }
    }
    put_cells(L.s, sv);
    put_cells(L.gp, gv);
    put_g(ov);
    __syncthreads();
    if (A.gp_prev != nullptr) conv_t(r0);
    float w1a[4][8];   // [t][kc] = W1[16t + n][feature(kc, g)]
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int kc = 0; kc < 8; ++kc) w1a[t][kc] = L.w1t[feature_of(kc, g) * kLd1 + 16 * t + n];
    if constexpr (NDIM == 2) clear();
    __syncthreads();

    const Rect own = region(0);
    float *const patch = L.patch[wave];
    const uint32_t state_bytes = (uint32_t)(cells * C * 4);
    for (int s = 0; s < k; ++s) {
        const bool last = s + 1 == k;
        float4 nv[kLoads];
        if (!last) load_cells(state_of(s + 1), nv);
        const Rect r = region(k - 1 - s);
        const int w = r.xb - r.xa;
        const int ow = own.xb - own.xa, oh = own.yb - own.ya;
        const int n_own = NDIM == 3 ? 256 : ow * oh;
        const int top = (own.ya - r.ya) * w, bottom = (r.yb - own.yb) * w;
        const int side = w - ow;
        const int n_ring = NDIM == 3 ? 0 : top + bottom + oh * side;
        const int own_groups = (n_own + 15) / 16, groups = own_groups + (n_ring + 15) / 16;
        const uint32_t m_own = (65536u + ow - 1) / ow, m_w = (65536u + w - 1) / w,
                       m_side = side > 0 ? (65536u + side - 1) / side : 0;
        const Rsrc wp = make_rsrc(A.gpart, last ? state_bytes : 0u);
        const Rsrc wg = make_rsrc(A.gp, last ? state_bytes : 0u);

        for (int u = wave; u < groups; u += kBwWaves) {
            const bool is_own = u < own_groups;              // uniform in the wave
            int z = 0, y, x;
            bool valid;
            if constexpr (NDIM == 3) {
                const int i = u * 16 + n;
                z = z0 + i / 64;
                y = y0 + (i >> 3) % 8;
                x = x0 + i % 8;
                valid = z < A.dd && y < A.dh && x < A.dw;
                z = min(z, A.dd - 1);
                y = min(y, A.dh - 1);
                x = min(x, A.dw - 1);
            } else if (is_own) {
                const int i = min(u * 16 + n, n_own - 1);
                valid = u * 16 + n < n_own;
                const int yy = (int)(((uint32_t)i * m_own) >> 16);
                y = own.ya + yy;
                x = own.xa + i - yy * ow;
            } else {
                // the ring around the tile: rows above, rows below, sides
                const int j = (u - own_groups) * 16 + n;
                const int i = min(j, n_ring - 1);
                valid = j < n_ring;
                if (i < top + bottom) {
                    const int b = i < top ? i : i - top;
                    const int yy = (int)(((uint32_t)b * m_w) >> 16);
                    y = (i < top ? r.ya : own.yb) + yy;
                    x = r.xa + b - yy * w;
                } else {
                    const int b = i - top - bottom;
                    const int yy = (int)(((uint32_t)b * m_side) >> 16);
                    y = own.ya + yy;
                    const int c = b - yy * side;
                    x = c < own.xa - r.xa ? r.xa + c : own.xb + c - (own.xa - r.xa);
                }
            }
            const int p = at(z, y, x), pg = at_g(z, y, x);
            const float4 own_s = L.s[g][p];
            const float4 go = L.g[g][pg];
            const int row = NDIM == 3 ? (z - z0) * 8 + y - y0 : y - r0.ya;
            const uint64_t fw = L.fire[s][row];
            const int fsh = (int)((uint32_t)((z * A.dh + y) * A.dw + r0.xa) & 7u) + x - r0.xa;
            float f[8] = {own_s.x, own_s.y, own_s.z, own_s.w};
            {
                const float4 cb = L.kb[g];
                float pc[4] = {cb.x, cb.y, cb.z, cb.w};
#pragma unroll
                for (int t = 0; t < TAPS; ++t) {
                    const int dz = NDIM == 3 ? t / 9 - 1 : 0, dy = (t / 3) % 3 - 1, dx = t % 3 - 1;
                    const float4 v = L.s[g][p + dz * 100 + dy * hx + dx];
                    const float4 c = L.kw[t][g];
                    pc[0] = fmaf(c.x, v.x, pc[0]);
                    pc[1] = fmaf(c.y, v.y, pc[1]);
                    pc[2] = fmaf(c.z, v.z, pc[2]);
                    pc[3] = fmaf(c.w, v.w, pc[3]);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) f[4 + i] = pc[i];
            }
            // layer 1, recomputed
            v4f a[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float4 b = *reinterpret_cast<const float4 *>(&L.b1[16 * t + 4 * g]);
                a[t] = v4f{b.x, b.y, b.z, b.w};
            }
#pragma unroll
            for (int kc = 0; kc < 8; ++kc)
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    a[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w1a[t][kc], f[kc], a[t], 0, 0, 0);
            // gu, masked to the cells that fire (and to this tile's own cells)
            const float gq[4] = {go.x, go.y, go.z, go.w};
            const bool fires = valid && ((uint32_t)(fw >> fsh) & 1u);
            float gu[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) gu[i] = (4 * g + i >= NIN && fires) ? gq[i] : 0.f;
            v4f ga[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float4 c = *reinterpret_cast<const float4 *>(&L.w2t[(16 * t + n) * kLd2 + 4 * g]);
                const float cc[4] = {c.x, c.y, c.z, c.w};
                ga[t] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    ga[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(cc[i], gu[i], ga[t], 0, 0, 0);
            }
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) ga[t][i] = a[t][i] > 0.f ? ga[t][i] : 0.f;
            // [gS, gP] = W1^T ga
            v4f gsp[2];
            gsp[0] = gsp[1] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                float4 c[2];
#pragma unroll
                for (int ft = 0; ft < 2; ++ft)
                    c[ft] = *reinterpret_cast<const float4 *>(
                        &L.w1t[(16 * ft + n) * kLd1 + 16 * t + 4 * g]);
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int ft = 0; ft < 2; ++ft) {
                        const float cc = i == 0 ? c[ft].x : i == 1 ? c[ft].y : i == 2 ? c[ft].z : c[ft].w;
                        gsp[ft] = __builtin_amdgcn_mfma_f32_16x16x4f32(cc, ga[t][i], gsp[ft], 0, 0, 0);
                    }
            }
            const float4 gn = make_float4(gq[0] + gsp[0][0], gq[1] + gsp[0][1], gq[2] + gsp[0][2],
                                          gq[3] + gsp[0][3]);
            if (valid) {
                L.gp[g][p] = make_float4(gsp[1][0], gsp[1][1], gsp[1][2], gsp[1][3]);
                if (!last) L.g[g][pg] = gn;
            }
            if (is_own) {
                const uint32_t off =
                    valid ? (uint32_t)((z * A.dh + y) * A.dw + x) * (C * 4) + 16 * g : kOut;
                const v4u o1 = {__float_as_uint(gn.x), __float_as_uint(gn.y), __float_as_uint(gn.z),
                                __float_as_uint(gn.w)};
                const v4u o2 = {__float_as_uint(gsp[1][0]), __float_as_uint(gsp[1][1]),
                                __float_as_uint(gsp[1][2]), __float_as_uint(gsp[1][3])};
                __builtin_amdgcn_raw_buffer_store_b128(o1, wp, off, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b128(o2, wg, off, 0, 0);

                // weight gradients of the 16 cells: gu (and with it ga and gP)
                // is 0 in lanes without a cell
                float *const mine = patch + n * kPatch + 4 * g;
                auto put = [&](int at_col, const v4f &v) {
                    *reinterpret_cast<float4 *>(mine + at_col) = make_float4(v[0], v[1], v[2], v[3]);
                };
                auto get = [&](int col, int c4) { return patch[(4 * c4 + g) * kPatch + col + n]; };
                // dW1: f at columns 0 .. 31, two hidden tiles of ga at 32 .. 63
                put(0, v4f{f[0], f[1], f[2], f[3]});
                put(16, v4f{f[4], f[5], f[6], f[7]});
                float fb[2][4];
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    put(32, ga[2 * half]);
                    put(48, ga[2 * half + 1]);
                    __builtin_amdgcn_wave_barrier();
                    if (half == 0)
#pragma unroll
                        for (int ft = 0; ft < 2; ++ft)
#pragma unroll
                            for (int c4 = 0; c4 < 4; ++c4) fb[ft][c4] = get(16 * ft, c4);
#pragma unroll
                    for (int c4 = 0; c4 < 4; ++c4)
#pragma unroll
                        for (int t = 0; t < 2; ++t) {
                            const float av = get(32 + 16 * t, c4);
#pragma unroll
                            for (int ft = 0; ft < 2; ++ft)
                                dw1[2 * half + t][ft] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                                    av, fb[ft][c4], dw1[2 * half + t][ft], 0, 0, 0);
                        }
                    __builtin_amdgcn_wave_barrier();
                }
                // dW2: gu at columns 0 .. 15, all of h at 16 .. 79
                put(0, v4f{gu[0], gu[1], gu[2], gu[3]});
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    put(16 + 16 * t, v4f{fmaxf(a[t][0], 0.f), fmaxf(a[t][1], 0.f),
                                         fmaxf(a[t][2], 0.f), fmaxf(a[t][3], 0.f)});
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int c4 = 0; c4 < 4; ++c4) {
                    const float av = get(0, c4);
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        dw2[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, get(16 + 16 * t, c4),
                                                                      dw2[t], 0, 0, 0);
                }
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int t = 0; t < 4; ++t) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) db1[t][i] += ga[t][i];
                    dcb[t] += gsp[1][t];
                }
                if constexpr (NDIM == 2) {
#pragma unroll
                    for (int t = 0; t < 9; ++t) {
                        const float4 v = L.s[g][p + (t / 3 - 1) * hx + t % 3 - 1];
                        dcw[t][0] = fmaf(gsp[1][0], v.x, dcw[t][0]);
                        dcw[t][1] = fmaf(gsp[1][1], v.y, dcw[t][1]);
                        dcw[t][2] = fmaf(gsp[1][2], v.z, dcw[t][2]);
                        dcw[t][3] = fmaf(gsp[1][3], v.w, dcw[t][3]);
                    }
                }
            }
        }
        if (!last) {
            __syncthreads();
            put_cells(L.s, nv);
            conv_t(region(k - 2 - s));
            __syncthreads();
        }
    }

    // 3D dconv_w: a job is a channel quad, a (dz, dy) pair of taps and a share
    // of the tile's 32 rows of 8 cells, the three dx taps from a sliding
    // window; kShare lanes per job (36 jobs on threads 0 .. 287)
    if constexpr (NDIM == 3) {
        __syncthreads();
        if (kjob < 36) {
            const int q = kjob & 3, dz = kjob / 12 - 1, dy = (kjob / 4) % 3 - 1;
            for (int row = (int)threadIdx.x % kShare; row < 32; row += kShare) {
                const int z = z0 + row / 8, y = y0 + row % 8;
                if (z >= A.dd || y >= A.dh) continue;
                const int pr = at(z, y, x0), ps = pr + dz * 100 + dy * hx;
                float4 v0 = L.s[q][ps - 1], v1 = L.s[q][ps];
                const int xn = min(8, A.dw - x0);
                for (int i = 0; i < xn; ++i) {
                    const float4 v2 = L.s[q][ps + i + 1], gpv = L.gp[q][pr + i];
                    const float4 vs[3] = {v0, v1, v2};
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        kacc[d][0] = fmaf(gpv.x, vs[d].x, kacc[d][0]);
                        kacc[d][1] = fmaf(gpv.y, vs[d].y, kacc[d][1]);
                        kacc[d][2] = fmaf(gpv.z, vs[d].z, kacc[d][2]);
                        kacc[d][3] = fmaf(gpv.w, vs[d].w, kacc[d][3]);
                    }
                    v0 = v1;
                    v1 = v2;
                }
            }
        }
    }
    }

    if constexpr (NDIM == 3) {
#pragma unroll
        for (int d = 0; d < 3; ++d)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int m = 1; m < kShare; m *= 2) kacc[d][i] += __shfl_xor(kacc[d][i], m);
    }

    // ---- the block's row: the waves' sums added in wave order ----
    __syncthreads();
    Sums &M = sh.s;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int ft = 0; ft < 2; ++ft)
                M.dw[wave][(16 * t + 4 * g + i) * 2 * C + 16 * ft + n] = dw1[t][ft][i];
            M.dw[wave][2 * C * H + (4 * g + i) * H + 16 * t + n] = dw2[t][i];
        }
    // sums over the 16 cells of a lane group
    auto over_cells = [&](float v) {
        // rotations within a row of 16 lanes (DPP row_ror 8, 4, 2, 1)
        auto ror = [](float x, auto c) {
            return __int_as_float(__builtin_amdgcn_update_dpp(
                0, __float_as_int(x), 0x120 + decltype(c)::value, 0xf, 0xf, false));
        };
        v += ror(v, std::integral_constant<int, 8>{});
        v += ror(v, std::integral_constant<int, 4>{});
        v += ror(v, std::integral_constant<int, 2>{});
        v += ror(v, std::integral_constant<int, 1>{});
        return v;
    };
#pragma unroll
    for (int t = 0; t < 4; ++t) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float v = over_cells(db1[t][i]);
            if (n == 0) M.db[wave][16 * t + 4 * g + i] = v;
        }
        const float v = over_cells(dcb[t]);
        if (n == 0) M.db[wave][H + 4 * g + t] = v;
    }
    if constexpr (NDIM == 2) {
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float v = over_cells(dcw[t][i]);
                if (n == 0) M.dk[wave][(4 * g + i) * 9 + t] = v;
            }
    }
    __syncthreads();
    float *const out = A.partial + (int64_t)blockIdx.x * G::N;
    for (int o = threadIdx.x; o < (NDIM == 2 ? G::N : G::CW); o += kBwThreads) {
        float v = 0.f;
#pragma unroll
        for (int wv2 = 0; wv2 < kBwWaves; ++wv2)
            v += o < G::B1 ? M.dw[wv2][o] : o < G::CW ? M.db[wv2][o - G::B1] : M.dk[wv2][o - G::CW];
        out[o] = A.accumulate ? out[o] + v : v;
    }
    if constexpr (NDIM == 3) {
        if (kjob < 36 && threadIdx.x % kShare == 0) {
            const int q = kjob & 3, t0 = (kjob / 4) * 3;
#pragma unroll
            for (int d = 0; d < 3; ++d)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float *const o = out + G::CW + (4 * q + i) * 27 + t0 + d;
                    *o = A.accumulate ? *o + kacc[d][i] : kacc[d][i];
                }
        }
    }
}

constexpr int64_t kPlanCus = 256;

int64_t tiles_of(const StepArgs &a, int tile) {
    if (a.ndim == 3) return (a.ext.d + 3) / 4 * ((a.ext.h + 7) / 8) * ((a.ext.w + 7) / 8);
    return (a.ext.h + tile - 1) / tile * ((a.ext.w + tile - 1) / tile);
}
// Blocks of a launch: in 3D the tiles divided evenly over as few rounds as one
// block per CU of a full MI355X gives.  A block adds up its tiles' weight
// gradients in fp32 (the rows are added in fp64), so from kBw3dTiles tiles a
// block on the launch is that many blocks per CU, one after another.  With all
// tiles of a CU in one sum (38 of them in 24 x 320 x 320 cells, 100 in 40 x 400
// x 400), the gradients of states of one sign were 1 to 4% further from 64 bits
// than those of 64-cell blocks (dconv_w 1.60e-7 and 1.55e-7), with at most eight
// they are as near.
constexpr int64_t kBw3dTiles = 8;
int64_t blocks_of(const StepArgs &a, int64_t tiles) {
    if (a.ndim == 2) return tiles;
    const int64_t rounds = (tiles + kPlanCus - 1) / kPlanCus;
    const int64_t sums = (rounds + kBw3dTiles - 1) / kBw3dTiles;   // blocks per CU
    const int64_t per_block = (rounds + sums - 1) / sums;
    return (tiles + per_block - 1) / per_block;
}

// Time model of a 2D level's launches on T x T tiles, in us: a launch with its
// set-up and the sums at its end, a tile's loads, per step the barriers and
// the transposed convolution, and per 4 groups of 16 cells (one per SIMD; 128
// fp32 MFMAs of 32 cycles for own cells, 80 for the ring) the matrix-core
// time.  Measured per step, model in brackets: 320^2 with T 20, k 2: 24.1 us
// (25.3), T 16, k 3: 33.6 (33.0); 160^2 with T 10, k 4: 11.9 (11.6), T 20, k 2:
// 26.0 (25.3); 40^2 with T 8, k 4: 8.2 (9.2), T 8, k 1: 14.1 (15.6).
constexpr double kBwLaunchUs = 7.5, kBwTileUs = 4.0, kBwStepUs = 1.6, kBwOwnUs = 2.45,
                 kBwRingUs = 1.5;
// A single 2D step below this size is faster on 64-cell blocks, which need not
// copy the weights and add up waves (a step's backward with its last two
// kernels, 64-cell blocks against these tiles: 33 x 61 cells 23.0 and 25.7 us,
// 100 x 128 24.3 and 27.1, 160^2 27.9 and 28.9, 200 x 220 38.0 and 36.4, 256^2
// 42.0 and 36.0, 320^2 62.0 and 45.3); two steps and more are not.
constexpr int64_t kBw2dOneStep = 32000;
// 3D levels take the tiles of 4 x 8 x 8 where a round of one block per CU has at
// least this many cells of its 65536 on average.  A round costs the same however
// full its tiles are (one plane of cells fills a quarter of a tile), 64-cell
// blocks cost by the cell.  A step of a ten-step training call, 64-cell blocks
// against these tiles, us: one round, 12 x 48 x 48 cells 36 and 44, 8 x 64 x 64
// 36 and 44, 16 x 48 x 48 45.8 and 45.1, 10 x 64 x 64 45.4 and 44.1, 24 x 48 x
// 48 57 and 51, 4 x 128 x 128 54 and 46; two, 5 x 96 x 96 53 and 61, 6 x 112 x
// 112 68.5 and 67.3, 3 x 160 x 160 83 and 67, 12 x 96 x 96 86 and 71; three, 2 x
// 200 x 200 67 and 81, 7 x 131 x 129 109 and 95; four, 256 x 256 85 and 91, 24 x
// 96 x 96 152 and 118; ten, 24 x 160 x 160 410 and 266.
constexpr int64_t kBw3dRoundCells = 36000;

double bwd_cost(int64_t h, int64_t w, int steps, int tile, int launches) {
    const int64_t tiles = (h + tile - 1) / tile * ((w + tile - 1) / tile);
    const double rounds = (double)((tiles + kPlanCus - 1) / kPlanCus);
    auto one = [&](int k) {
        double t = kBwTileUs;
        const int64_t own = std::min<int64_t>(h, tile) * std::min<int64_t>(w, tile);
        for (int e = 0; e < k; ++e) {
            const int64_t all = std::min<int64_t>(h, tile + 2 * e) * std::min<int64_t>(w, tile + 2 * e);
            const int64_t og = (own + 15) / 16, rg = (all - own + 15) / 16;
            const int64_t turns = (og + rg + 3) / 4, oturns = (og + 3) / 4;
            t += kBwStepUs + kBwOwnUs * (double)oturns + kBwRingUs * (double)(turns - oturns);
        }
        return kBwLaunchUs + rounds * t;
    };
    const int more = steps % launches;
    return (more ? more * one(steps / launches + 1) : 0.0) +
           (launches - more) * one(steps / launches);
}

}  // namespace

bool bwd_block_plan(const StepArgs &a, int steps, int64_t max_blocks, BwdBlockPlan *plan) {
    if (a.channels != 16 || a.hidden != 64 || steps < 1) return false;
    // 32-bit byte offsets into a state
    if (a.ext.cells() > (int64_t(1) << 32) / 64 - 1) return false;
    if (a.ndim == 3) {
        const int64_t tiles = tiles_of(a, 8), rounds = (tiles + kPlanCus - 1) / kPlanCus;
        if (a.ext.cells() < kBw3dRoundCells * rounds || blocks_of(a, tiles) > max_blocks)
            return false;
        plan->tile = 8;
        plan->launches = steps;
        return true;
    }
    if (steps == 1 && a.ext.cells() < kBw2dOneStep) return false;
    double best = 1e30;
    plan->launches = 0;
    for (int tile : {6, 8, 10, 12, 14, 16, 18, 20, 22}) {
        if (blocks_of(a, tiles_of(a, tile)) > max_blocks) continue;   // rows of the workspace
        int last = 0;
        for (int k = std::min({(kBwRegion - tile) / 2, kBwMaxSteps, steps}); k >= 1; --k) {
            const int launches = (steps + k - 1) / k;
            if (launches == last) continue;
            last = launches;
            const double c = bwd_cost(a.ext.h, a.ext.w, steps, tile, launches);
            if (c < best) {
                best = c;
                plan->tile = tile;
                plan->launches = launches;
            }
        }
    }
    return plan->launches > 0;
}

int64_t bwd_block_rows(const StepArgs &a, const BwdBlockPlan &plan) {
    return blocks_of(a, tiles_of(a, plan.tile));
}

hipError_t launch_bwd_block(const StepArgs &a, const BwdBlockPlan &plan, int steps,
                            const float *state, const float *gout, const float *gp_prev,
                            float *gpart, float *gp, float *partial, bool accumulate,
                            hipStream_t stream) {
    const int64_t tiles = tiles_of(a, plan.tile), blocks = blocks_of(a, tiles);
    if (tiles == 0) return hipSuccess;
    if (tiles > INT32_MAX || steps < 1 || steps > (a.ndim == 3 ? 1 : kBwMaxSteps) ||
        (a.ndim == 2 && plan.tile + 2 * steps > kBwRegion))
        return hipErrorInvalidValue;
    BwArgs b{};
    b.states = state;
    b.gout = gout;
    b.gp_prev = gp_prev;
    b.gpart = gpart;
    b.gp = gp;
    b.partial = partial;
    b.conv_w = a.w.conv_w;
    b.conv_b = a.w.conv_b;
    b.w1 = a.w.w1;
    b.b1 = a.w.b1;
    b.w2 = a.w.w2;
    b.seed = a.seed;
    b.threshold = a.threshold;
    b.dd = (int)a.ext.d;
    b.dh = (int)a.ext.h;
    b.dw = (int)a.ext.w;
    b.tile = plan.tile;
    b.tiles = (int)tiles;
    const int t = a.ndim == 3 ? 8 : plan.tile;
    b.tiles_x = (int)((a.ext.w + t - 1) / t);
    b.tiles_y = (int)((a.ext.h + t - 1) / t);
    b.steps = steps;
    b.accumulate = accumulate ? 1 : 0;
    b.level = a.level;
    b.step = a.step;
    b.batch = a.batch;
    auto kern = a.ndim == 2 ? (a.n_in == 1 ? bwd_block<2, 1> : bwd_block<2, 3>)
                            : (a.n_in == 1 ? bwd_block<3, 1> : bwd_block<3, 3>);
    kern<<<(unsigned)blocks, kBwThreads, 0, stream>>>(b);
    return hipGetLastError();
}

}  // namespace octnca
