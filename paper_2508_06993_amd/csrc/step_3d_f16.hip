// NCA step for fp16 3D states (video), C = 16, H = 64, with the perception and
// the MLP both on the matrix cores.
//
// A depthwise 3x3x3 convolution is no contraction over channels, but for one
// channel the outputs of a 2 x 8 block of cells (y, x) are a matrix product:
// 16 outputs x (3 planes x 4 rows x 10 columns of inputs), with a banded
// (Toeplitz) matrix of the 27 taps that is the same for every block.  A
// v_mfma_f32_16x16x32_f16 takes that matrix as A and one input plane's 4 rows x
// 8 columns of 16 blocks as B; a fourth one takes the two remaining columns of
// the three planes, and the bias.  So a channel of 256 cells costs 4 MFMAs (64
// cycles) where packed fp16 FMAs took 13.5 x 4 instructions a SIMD (864 cycles
// per 64 cells and 16 channels against 256), and the sums are fp32 now (the
// packed ones were rounded to fp16 after every tap).
//
// A block of 4 waves owns an 8 x 32 (y, x) column and a run of planes.  Wave w
// computes the perception of channels 4w .. 4w+3 for all 256 cells of a plane,
// leaves it in LDS, and runs the MLP (lane layout of step_mfma.hip) of its own
// 64 cells of the previous plane; the two are independent, so one block
// barrier per plane is enough.  The planes sit in LDS channel by channel (x
// contiguous: a B operand is one 16-byte read), four of them in a ring.  They
// come from memory cell by cell; neighbouring lanes hold neighbouring cells
// and exchange halves (DPP, v_perm) to write two cells of a channel at once.
//
// The zero entries of the banded matrix meet cells that are in a block's
// window but not in an output's stencil: an infinity there would turn the
// product into a NaN.  So each wave checks its perception for values that are
// not finite, and where there is one computes that plane's values tap by tap.
#include <algorithm>

#include "launch.h"
#include "step_common.h"

namespace octnca {

namespace {

constexpr int kTY = 8, kTX = 32;            // the block's cells of a plane
constexpr int kThreads3 = 256;
constexpr int kHaloRows = kTY + 2;
constexpr int kHaloCells = kTX + 2;
// LDS planes, channel by channel: 10 rows of 32 halves (halo columns 0 .. 31),
// then the rows' columns 32, 33.  A 16-byte read takes lanes 0-3, 12-15, 20-23
// and 24-27 (and so on) together; with rows of 64 bytes the window rows of
// those lanes' blocks fall on all the banks once (rows of 80 bytes measured 3
// conflicts a read).  Channels are 44 words mod 64 apart, for the writes (16
// cell pairs x 2 parities x 2 chunks of 8 channels) and the centre reads.
constexpr int kRow = 32;
constexpr int kTail = kHaloRows * kRow;
constexpr int kChan = kTail + 2 * kHaloRows + 4;
constexpr int kPlane = kC * kChan;
__device__ __forceinline__ int lds_at(int row, int col) {
    return col < 32 ? row * kRow + col : kTail + 2 * row + col - 32;
}
// perception: quad planes of 8-byte words, rows of 34 (the four blocks above
// each other that a write covers would otherwise share their banks)
constexpr int kPRow = kTX + 2;
constexpr int kPQuad = kTY * kPRow;
constexpr int kEvals = 32;                  // fire evaluations of a run
constexpr int kMaxRun = kEvals * 8;         // planes of a run (rows 8-aligned; else half)
constexpr int kBlocksPerCu3 = 2;
// a channel's taps in LDS: nine rows of three taps and a zero, then the bias
constexpr int kBias = 9 * 4, kTaps = kBias + 4;

typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef float v2f_ __attribute__((ext_vector_type(2)));

__device__ __forceinline__ h2 as_h2(uint32_t u) { return __builtin_bit_cast(h2, u); }
__device__ __forceinline__ uint32_t as_u32(h2 v) { return __builtin_bit_cast(uint32_t, v); }
// (mask & a) | (~mask & b) in one instruction (the compiler builds it from
// two ands, an and-or and the mask's complement)
__device__ __forceinline__ uint32_t bfi(uint32_t mask, uint32_t a, uint32_t b) {
    uint32_t r;
    asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(r) : "v"(mask), "v"(a), "v"(b));
    return r;
}

template <typename V> using Lds = __attribute__((address_space(3))) V;

struct Args3 {
    const __half *src;     // the level's state, or the coarse state (UP)
    __half *dst;
    const __half *img;     // the level's image (UP)
    uint8_t *seg;          // readout (SEG)
    const float *conv_w, *conv_b, *w1, *b1, *w2;
    uint64_t seed, threshold;
    int dd, dh, dw, tiles_x, tiles_y, items, zrun;
    int cdh, cdw, fz, fy, fx;
    uint32_t level, step, batch;
};

// UP: the first step of a level fused with the upsample + inject: src is the
// next coarser level's state (planes of cdh x cdw cells), upsampled by
// (fz, fy, fx), with the input channels from img.  SEG: the launch also writes
// the two-class readout of the state it stores (channel C - 1 > channel C - 2
// in the stored fp16 values, ties and NaNs 0).
template <int NIN, bool ALIGNED, bool UP, bool SEG>
__global__ __launch_bounds__(kThreads3, kBlocksPerCu3) void nca_step_3d_f16(const Args3 A) {
    __shared__ __align__(16) _Float16 ring[4][kPlane];       // plane z in slot z & 3
    __shared__ __align__(16) uint2 pbuf[2][4 * kPQuad];      // perception of plane z in z & 1
    __shared__ uint64_t fire_words[4][kEvals][8];
    __shared__ __align__(8) _Float16 cw[kC][kTaps];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15;
    const int g = lane >> 4;
    const int dd = A.dd, dh = A.dh, dw = A.dw;

    for (int i = threadIdx.x; i < kC * kTaps; i += kThreads3) {
        const int c = i / kTaps, t = i % kTaps, tap = t / 4 * 3 + t % 4;
        const float v = *(t < kBias ? A.conv_w + c * 27 + min(tap, 26) : A.conv_b + c);
        cw[c][t] = (_Float16)(t % 4 < 3 ? v : 0.f);
    }
    MlpF16 mlp;
    mlp.load(A.w1, A.b1, A.w2, n, g, NIN);
    mlp.pin_all();
    __syncthreads();
    // The banded matrices of the wave's channels.  Row n of A is output (oy,
    // ox) = (n / 8, n % 8) of a block; K slot j of lane group g is, in plane
    // dz (matrix dz), window row g and column j, and in the last matrix plane
    // j / 2, window row g and column 8 + j % 2 (slot 6 of lane group 0: the bias,
    // against 1).
    v8h am[4][4];
    {
        // A row of taps is 48 bits; a row of the matrix has them ox halves up
        // (choosing each element by compares took 0.6 us of a small volume's step:
        // 4 x 16 x 16 cells 9.4 us, now 8.6).
        const int oy = n >> 3, ox = n & 7;
        const int dy = g - oy, row = min(max(dy, 0), 2);
        const bool in = dy == row, high = ox >= 4;
        const int up = 16 * (ox & 3);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v4u last = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                const uint2 w = *reinterpret_cast<const uint2 *>(cw[4 * wave + q] + 4 * (3 * m + row));
                const uint32_t w0 = in ? w.x : 0u, w1 = in ? w.y : 0u;
                const uint64_t taps = (uint64_t)w1 << 32 | w0;
                const uint64_t a = taps << up, over = (taps >> 1) >> (63 - up);
                const v4u r = {high ? 0u : (uint32_t)a, high ? 0u : (uint32_t)(a >> 32),
                               high ? (uint32_t)a : (uint32_t)over,
                               high ? (uint32_t)(a >> 32) : (uint32_t)(over >> 32)};
                am[q][m] = __builtin_bit_cast(v8h, r);
                // columns 8, 9: taps 1 and 2 of output 7, tap 2 of output 6
                last[m] = ox == 7 ? __builtin_amdgcn_alignbyte(w1, w0, 2) : ox == 6 ? w1 : 0u;
            }
            const uint32_t bias = *reinterpret_cast<const uint32_t *>(cw[4 * wave + q] + kBias) & 0xffffu;
            last[3] = g == 0 ? bias : 0u;
            am[q][3] = __builtin_bit_cast(v8h, last);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int m = 0; m < 4; ++m) pin(am[q][m]);
    }
    float one = 1.f;
    uint32_t one_zero = 0x00003c00u;   // fp16 (1, 0): the bias's K slot
    pin(one);
    pin(one_zero);
    // fire evaluations: lane -> (plane, row of the wave's two, 8-cell block);
    // ALIGNED (w % 8 == 0) makes the bit offsets of a lane's cells constants
    constexpr int opr = ALIGNED ? 4 : 8;
    constexpr int lg_opr = ALIGNED ? 2 : 3;
    constexpr int planes_per_eval = 64 / (2 * opr);
    constexpr uint32_t kCellBytes = kC * 2;
    const uint32_t row_bytes = (uint32_t)dw * kCellBytes;

    // Loads of a plane's halo rows: load i of the block (i = thread + 256 k) is
    // chunk (i / 2) % 2 (8 channels) of cell 2 (i / 4 % 17) + i % 2 of row
    // i / 68, so four lanes read 64 contiguous bytes.
    constexpr int kLoadsAll = kHaloRows * kHaloCells * 2;
    constexpr int kLoads = (kLoadsAll + kThreads3 - 1) / kThreads3;
    struct Regs {
        uint4 v[kLoads];
    };
    constexpr int kImgAll = kHaloRows * kHaloCells * NIN;
    constexpr int kImg = (kImgAll + kThreads3 - 1) / kThreads3;
    uint32_t lofs[kLoads];             // byte offsets in the tile's rows
    uint32_t iofs[UP ? kImg : 1];      // image (UP)
    uint32_t im[UP ? kImg : 1];
    int y0 = 0, x0 = 0;
    auto rows_of = [&](int z, bool active) {
        const int base = max(y0 - 1, 0);
        return active && z >= 0 && z < dd ? max(0, min(y0 - 1 + kHaloRows, dh) - base) : 0;
    };
    auto issue = [&](Regs &r, int z, bool active) {
        const int base = max(y0 - 1, 0);
        const int rows = rows_of(z, active);
        Rsrc s;
        if constexpr (UP) {
            const int cbase = base / A.fy;
            const int crows = rows > 0 ? (base + rows - 1) / A.fy - cbase + 1 : 0;
            s = make_rsrc(A.src + ((int64_t)(max(z, 0) / A.fz) * A.cdh + cbase) * A.cdw * kC,
                          (uint32_t)crows * (uint32_t)A.cdw * kCellBytes);
            const Rsrc si = make_rsrc(A.img + ((int64_t)max(z, 0) * dh + base) * dw * NIN,
                                      (uint32_t)rows * (uint32_t)dw * NIN * 2u);
#pragma unroll
            for (int k = 0; k < kImg; ++k)
                im[k] = __builtin_amdgcn_raw_buffer_load_b16(si, iofs[k], 0, 0);
        } else {
            s = make_rsrc(A.src + ((int64_t)max(z, 0) * dh + base) * dw * kC,
                          (uint32_t)rows * row_bytes);
        }
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {
            const v4u x = __builtin_amdgcn_raw_buffer_load_b128(s, lofs[k], 0, 0);
            r.v[k] = make_uint4(x[0], x[1], x[2], x[3]);
        }
    };
    // LDS address (halves) of the lane's writes: channel 8 chunk + parity of
    // its cell pair; the k-th word of a chunk goes 2 k channels further
    uint32_t wofs[kLoads];
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {
        const int i = (int)threadIdx.x + kThreads3 * k;
        const int row = i / 68, rem = i % 68;
        wofs[k] = (uint32_t)((8 * ((rem >> 1) & 1) + (rem & 1)) * kChan + lds_at(row, 2 * (rem >> 2)));
    }
    // v_perm selectors: the even lane joins the low halves (its cell first),
    // the odd lane the high halves (its cell second)
    const uint32_t sel = lane & 1 ? 0x03020706u : 0x05040100u;
    auto commit = [&](const Regs &r, int z) {
        _Float16 *slot = ring[z & 3];
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {
            const uint32_t own[4] = {r.v[k].x, r.v[k].y, r.v[k].z, r.v[k].w};
            uint32_t out[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                // quad_perm [1, 0, 3, 2]: the other cell of the pair
                const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(
                    0, (int)own[c], 0xb1, 0xf, 0xf, false);
                out[c] = __builtin_amdgcn_perm(other, own[c], sel);
            }
            if (kThreads3 * (k + 1) <= kLoadsAll || (int)threadIdx.x + kThreads3 * k < kLoadsAll)
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    *reinterpret_cast<uint32_t *>(slot + wofs[k] + 2 * c * kChan) = out[c];
        }
    };
    // UP: the image values over the input channels that another lane wrote
    auto commit_image = [&](int z) {
        if constexpr (UP) {
            __syncthreads();
            _Float16 *slot = ring[z & 3];
#pragma unroll
            for (int k = 0; k < kImg; ++k) {
                const int i = (int)threadIdx.x + kThreads3 * k;
                const int cell = i / NIN, c = i % NIN;
                if (i < kImgAll)
                    slot[c * kChan + lds_at(cell / kHaloCells, cell % kHaloCells)] =
                        __builtin_bit_cast(_Float16, (unsigned short)im[k]);
            }
        }
    };

    // Perception of plane z from planes z - 1, z, z + 1 of the ring.  Lane
    // (n, g): block (by, bx) = (n / 4, n % 4), window row g.
    const int by = n >> 2, bx = n & 3;
    const int b_at = (2 * by + g) * kRow + 8 * bx;           // columns 0 .. 7 of row g
    const int e_at = lds_at(2 * by + g, 8 * bx + 8);         // columns 8, 9
    int c_at[4];                       // the lane's cells in an MLP group, channel 4g
#pragma unroll
    for (int grp = 0; grp < 4; ++grp)
        c_at[grp] = 4 * g * kChan + lds_at(2 * wave + (grp >> 1) + 1, (grp & 1) * 16 + n + 1);
#pragma unroll
    for (int grp = 0; grp < 4; ++grp) pin(c_at[grp]);
    const int p_at = (2 * by + (g >> 1)) * kPRow + 8 * bx + 4 * (g & 1);
    auto perceive = [&](int z) -> bool {
        const _Float16 *pl[3] = {ring[(z + 3) & 3] + 4 * wave * kChan,
                                 ring[z & 3] + 4 * wave * kChan,
                                 ring[(z + 1) & 3] + 4 * wave * kChan};
        v4f acc[4];
        v8h b[3][4];
        uint32_t e[4][3];
        auto read = [&](int m) {
#pragma unroll
            for (int q = 0; q < 4; ++q) b[m][q] = *reinterpret_cast<const v8h *>(pl[m] + q * kChan + b_at);
        };
        // two planes of operands in flight ahead of the MFMAs that take them
        read(0);
        read(1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_f16(am[q][0], b[0][q],
                                                            v4f{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        read(2);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_f16(am[q][1], b[1][q], acc[q], 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int m = 0; m < 3; ++m)
                // (volatile: reads of two channels merged into one would leave
                // the words of an operand in registers apart, a move each)
                e[q][m] = *(const volatile Lds<uint32_t> *)(pl[m] + q * kChan + e_at);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_f16(am[q][2], b[2][q], acc[q], 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const v4u ev = {e[q][0], e[q][1], e[q][2], one_zero};
            acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_f16(am[q][3], __builtin_bit_cast(v8h, ev),
                                                            acc[q], 0, 0, 0);
        }
        // four consecutive cells of the wave's channel quad, rounded to fp16
        uint32_t o[4][2];
        h2 bad = {(_Float16)0.f, (_Float16)0.f};
        const h2 zero = bad;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const h2 v = __builtin_convertvector(v2f_{acc[2 * k][i], acc[2 * k + 1][i]}, h2);
                o[i][k] = as_u32(v);
                bad = __builtin_elementwise_fma(v, zero, bad);   // NaN unless finite
            }
        uint2 *out = pbuf[z & 1] + wave * kPQuad + p_at;
        *reinterpret_cast<uint4 *>(out) = make_uint4(o[0][0], o[0][1], o[1][0], o[1][1]);
        *reinterpret_cast<uint4 *>(out + 2) = make_uint4(o[2][0], o[2][1], o[3][0], o[3][1]);
        return (float)bad[0] == 0.f && (float)bad[1] == 0.f;
    };
    // Some input or sum of plane z is not finite: the wave's channels again, each
    // output from its own 27 cells.  Lane (n, g) takes channel g of the wave's and
    // all of block n, so a row of its window is two reads and serves two rows of
    // outputs (two taps a dot product of fp16 values, fp32 sums); the four lanes
    // of a block then exchange halves for the usual writes.  A 48 x 120 x 216
    // level of diverged states takes 58 us a step (131 with four neighbouring
    // cells a lane and a read per tap and cell: bound by those reads), finite
    // states, and one infinite cell among them, 34.
    auto perceive_exact = [&](int z) {
        // addresses from here: hoisted, they would hold registers of the plane loop
        int nn = n, gg = g;
        pin(nn);
        pin(gg);
        const int c = 4 * wave + gg, y = 2 * (nn >> 2), x = 8 * (nn & 3);
        const int body = c * kChan + y * kRow + x, tail = c * kChan + lds_at(y, x + 8);
        const int tail_row = x + 8 < 32 ? kRow : 2;
        float sum[2][8];
#pragma unroll
        for (int oy = 0; oy < 2; ++oy)
#pragma unroll
            for (int ox = 0; ox < 8; ++ox) sum[oy][ox] = (float)cw[c][kBias];
#pragma unroll 1
        for (int m = 0; m < 3; ++m) {
            const _Float16 *pl = ring[(z + m + 3) & 3];
            uint4 v8[4];
            uint32_t v2[4];
            uint2 w[3];      // taps 0 and 1 of a row, and tap 2
#pragma unroll
            for (int i = 0; i < 3; ++i)
                w[i] = *reinterpret_cast<const uint2 *>(cw[c] + 4 * (3 * m + i));
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                v8[r] = *reinterpret_cast<const uint4 *>(pl + body + r * kRow);
                v2[r] = *reinterpret_cast<const uint32_t *>(pl + tail + r * tail_row);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                // cells 2 i, 2 i + 1 and 2 i + 1, 2 i + 2 of the row
                const uint32_t even[5] = {v8[r].x, v8[r].y, v8[r].z, v8[r].w, v2[r]};
                uint32_t odd[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) odd[i] = __builtin_amdgcn_alignbyte(even[i + 1], even[i], 2);
#pragma unroll
                for (int oy = 0; oy < 2; ++oy) {
                    const int dy = r - oy;
                    if (dy < 0 || dy > 2) continue;
#pragma unroll
                    for (int ox = 0; ox < 8; ++ox) {
                        const uint32_t v01 = ox & 1 ? odd[ox / 2] : even[ox / 2];
                        sum[oy][ox] = __builtin_amdgcn_fdot2(as_h2(w[dy].x), as_h2(v01), sum[oy][ox], false);
                        sum[oy][ox] = fmaf((float)as_h2(w[dy].y)[0],
                                           (float)as_h2(even[ox / 2 + 1])[ox & 1], sum[oy][ox]);
                    }
                }
            }
        }
        // lane g: channel g of cells 4 q .. 4 q + 3 (q = 0 .. 3) -> channels 0 .. 3 of
        // cells 4 g .. 4 g + 3, two cells a word
        uint32_t o[4][2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            uint32_t q[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float *f = &sum[i >> 1][4 * (i & 1) + 2 * k];
                q[i] = as_u32(__builtin_convertvector(v2f_{f[0], f[1]}, h2));
            }
            const auto a = __builtin_amdgcn_permlane32_swap(q[0], q[2], false, false);
            const auto b = __builtin_amdgcn_permlane32_swap(q[1], q[3], false, false);
            const auto c01 = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
            const auto c23 = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
            o[2 * k][0] = __builtin_amdgcn_perm(c01[1], c01[0], 0x05040100u);
            o[2 * k][1] = __builtin_amdgcn_perm(c23[1], c23[0], 0x05040100u);
            o[2 * k + 1][0] = __builtin_amdgcn_perm(c01[1], c01[0], 0x07060302u);
            o[2 * k + 1][1] = __builtin_amdgcn_perm(c23[1], c23[0], 0x07060302u);
        }
        uint2 *out = pbuf[z & 1] + wave * kPQuad + (y + (gg >> 1)) * kPRow + x + 4 * (gg & 1);
        *reinterpret_cast<uint4 *>(out) = make_uint4(o[0][0], o[0][1], o[1][0], o[1][1]);
        *reinterpret_cast<uint4 *>(out + 2) = make_uint4(o[2][0], o[2][1], o[3][0], o[3][1]);
    };

    const int64_t span = ((int64_t)A.items + gridDim.x - 1) / gridDim.x * gridDim.x;
    for (int64_t u = blockIdx.x; u < span; u += gridDim.x) {
        const int64_t it = xcd_item(u, (int)gridDim.x);
        if (it >= A.items) continue;                       // uniform over the block
        const int tiles = A.tiles_x * A.tiles_y;
        const int zr = (int)it / tiles;
        const int rest = (int)it - zr * tiles;
        const int ty = rest / A.tiles_x;
        y0 = ty * kTY;
        x0 = (rest - ty * A.tiles_x) * kTX;
        const int z_begin = zr * A.zrun;
        const int z_end = min(dd, z_begin + A.zrun);
        {
            const int base = max(y0 - 1, 0);
#pragma unroll
            for (int k = 0; k < kLoads; ++k) {
                const int i = (int)threadIdx.x + kThreads3 * k;
                const int row = i / 68, rem = i % 68;
                const int gy = y0 - 1 + row, gx = x0 - 1 + 2 * (rem >> 2) + (rem & 1);
                const bool ok = i < kLoadsAll && gy >= 0 && gx >= 0 && gx < dw;
                const uint32_t chunk = (uint32_t)((rem >> 1) & 1) * 16u;
                uint32_t off;
                if constexpr (UP)
                    off = (uint32_t)(max(gy, 0) / A.fy - base / A.fy) * ((uint32_t)A.cdw * kCellBytes) +
                          (uint32_t)(max(gx, 0) / A.fx) * kCellBytes + chunk;
                else
                    off = (uint32_t)(gy - base) * row_bytes + (uint32_t)gx * kCellBytes + chunk;
                lofs[k] = ok ? off : kOut;
            }
            if constexpr (UP) {
#pragma unroll
                for (int k = 0; k < kImg; ++k) {
                    const int i = (int)threadIdx.x + kThreads3 * k;
                    const int cell = i / NIN;
                    const int gy = y0 - 1 + cell / kHaloCells, gx = x0 - 1 + cell % kHaloCells;
                    const bool ok = i < kImgAll && gy >= 0 && gx >= 0 && gx < dw;
                    iofs[k] = ok ? ((uint32_t)(gy - base) * (uint32_t)dw + (uint32_t)gx) * (NIN * 2u) +
                                       (uint32_t)(i % NIN) * 2u
                                 : kOut;
                }
            }
        }
        // store offsets of the lane's 4 cells within an output plane's tile rows
        uint32_t offs[4];
#pragma unroll
        for (int grp = 0; grp < 4; ++grp) {
            const int x = x0 + (grp & 1) * 16 + n;
            offs[grp] = x < dw ? (uint32_t)(2 * wave + (grp >> 1)) * row_bytes +
                                     (uint32_t)x * kCellBytes + 8u * g
                               : kOut;
        }

        // planes z_begin - 1 .. z_begin + 2 into the ring, the fire evaluations
        // of the run while the first one loads, the first plane's perception
        Regs r;
        __syncthreads();                 // the previous item is done with the ring
        issue(r, z_begin - 1, true);
        for (int e = 0; z_begin + e * planes_per_eval < z_end; ++e) {
            const int zo = z_begin + e * planes_per_eval;
            const int zz = min(zo + (lane >> (lg_opr + 1)), dd - 1);
            const uint64_t row =
                (uint64_t)zz * dh + (uint64_t)(y0 + 2 * wave + ((lane >> lg_opr) & 1));
            const FireBallots fb = fire_ballots(((row * dw + x0) >> 3) + (lane & (opr - 1)), A.step,
                                                A.level, A.batch, A.seed, A.threshold);
            uint64_t word = fb.w[0];
#pragma unroll
            for (int b = 1; b < 8; ++b) word = (lane & 7) == b ? fb.w[b] : word;
            fire_words[wave][e][lane & 7] = word;
        }
#pragma unroll 1
        for (int z = z_begin - 1; z <= z_begin + 1; ++z) {
            commit(r, z);
            commit_image(z);
            issue(r, z + 1, z + 1 <= z_end);
        }
        __syncthreads();
        if (__ballot(!perceive(z_begin)) != 0) perceive_exact(z_begin);
        commit(r, z_begin + 2);
        commit_image(z_begin + 2);
        issue(r, z_begin + 3, z_begin + 3 <= z_end);
        __syncthreads();

        for (int z = z_begin; z < z_end; ++z) {
            // the next plane's perception (past the run's end it is not used)
            const bool finite = perceive(z + 1);

            const int zrel = z - z_begin;
            const int phase = zrel & (planes_per_eval - 1);
            const uint64_t *fwe = fire_words[wave][zrel / planes_per_eval];
            const int slot0 = 2 * phase;
            const Rsrc wr = make_rsrc(A.dst + ((int64_t)z * dh + y0) * dw * kC,
                                      (uint32_t)min(kTY, dh - y0) * row_bytes);
            const _Float16 *own = ring[z & 3];
            const uint2 *pp = pbuf[z & 1] + g * kPQuad + 2 * wave * kPRow + n;
            // ALIGNED: the bits of the lane's 4 cells of this plane, at 2 grp
            uint32_t fw_lane = 0;
            if constexpr (ALIGNED) fw_lane = (uint32_t)(fwe[n & 7] >> (slot0 * opr + (n >> 3)));
#pragma unroll
            for (int grp = 0; grp < 4; ++grp) {
                const int at = c_at[grp];
                const h2 s01 = {own[at], own[at + kChan]};
                const h2 s23 = {own[at + 2 * kChan], own[at + 3 * kChan]};
                const v2u pv = *(const volatile Lds<v2u> *)(pp + (grp >> 1) * kPRow + (grp & 1) * 16);
                const h2 p01 = as_h2(pv[0]), p23 = as_h2(pv[1]);
                const v8h fh = {s01[0], s01[1], s23[0], s23[1], p01[0], p01[1], p23[0], p23[1]};
                v4f acc[4];
                mlp.layer1_h(fh, acc);
                const v4f u2 = mlp.layer2(acc);
                const int rr = grp >> 1;
                // all ones when the cell fires, else zero
                uint32_t keep_new;
                if constexpr (ALIGNED) {
                    // cell n of the group is cell n % 8 of block (grp & 1) * 2 + n / 8 of its
                    // row: bit (rr * opr + (grp & 1) * 2) of fw_lane, i.e. bit 2 grp
                    keep_new = (uint32_t)__builtin_amdgcn_sbfe((int)fw_lane, 2 * grp, 1);
                } else {
                    const int y = y0 + 2 * wave + rr, x = x0 + (grp & 1) * 16 + n;
                    const uint64_t idx = ((uint64_t)z * dh + y) * dw + x;
                    const uint64_t row_b0 = (((uint64_t)z * dh + y) * dw + x0) >> 3;
                    const uint64_t fw = fwe[idx & 7];
                    keep_new = (fw >> ((slot0 + rr) * opr + (int)((idx >> 3) - row_b0))) & 1 ? ~0u : 0u;
                }
                // state + update in fp32, rounded once to fp16 (u = +0 keeps an
                // input channel exactly); a cell that does not fire keeps its
                // stored bits
                // (as fmas with a register 1.0: one mixed-precision fma per value)
                const h2 n01 = {(_Float16)fmaf(one, u2[0], (float)s01[0]),
                                (_Float16)fmaf(one, u2[1], (float)s01[1])};
                const h2 n23 = {(_Float16)fmaf(one, u2[2], (float)s23[0]),
                                (_Float16)fmaf(one, u2[3], (float)s23[1])};
                const v2u out = {bfi(keep_new, as_u32(n01), as_u32(s01)),
                                 bfi(keep_new, as_u32(n23), as_u32(s23))};
                __builtin_amdgcn_raw_buffer_store_b64(out, wr, offs[grp], 0, 0);
                if constexpr (SEG) {
                    // lanes of quad 3: out[1] holds channels 14 (low) and 15 (high)
                    const h2 c1415 = as_h2(out[1]);
                    const int x = x0 + (grp & 1) * 16 + n;
                    const Rsrc sr = make_rsrc(A.seg + ((int64_t)z * dh + y0) * dw,
                                              (uint32_t)min(kTY, dh - y0) * dw);
                    const uint32_t so = g == 3 && x < dw ? (uint32_t)(2 * wave + rr) * dw + x : kOut;
                    __builtin_amdgcn_raw_buffer_store_b8(
                        (unsigned char)((float)c1415[1] > (float)c1415[0] ? 1 : 0), sr, so, 0, 0);
                }
            }

            if (__ballot(!finite) != 0) perceive_exact(z + 1);
            commit(r, z + 3);
            commit_image(z + 3);
            issue(r, z + 4, z + 4 <= z_end);
            __syncthreads();
        }
    }
}

template <int NIN, bool UP, bool SEG>
void launch3(const Args3 &b, int grid, hipStream_t stream) {
    if (b.dw % 8 == 0)
        nca_step_3d_f16<NIN, true, UP, SEG><<<grid, kThreads3, 0, stream>>>(b);
    else
        nca_step_3d_f16<NIN, false, UP, SEG><<<grid, kThreads3, 0, stream>>>(b);
}

}  // namespace

// Short runs spread a small level over the chip at the cost of streaming their
// halo planes again.  Where every item has a CU of its own a run costs 1.34 us
// a plane and little set-up; with two blocks a CU (and a round of items after
// the other) 3.9 us and 1.71 a plane (a fit to 900 launches: 75 levels, all run
// lengths; 6% rms).  So 256 items of one block per CU beat twice as many of
// half the length: counting only planes and block slots had taken runs of two
// on 14 x 243 x 64 cells, 17.6 us a step where runs of four take 14.7 (16 x 215
// x 64 17.1 and 14.8, 57 x 106 x 32 17.0 and 15.3, 24 x 96 x 96 16.5 and 14.9,
// 34 x 65 x 40 15.4 and 12.2).  On the 75 levels its choice is 0.3% off the best
// run length on average; that rule's was 11.7%.  Larger levels keep their runs.
int step_3d_f16_run(int64_t tiles, int64_t depth, int64_t cus, int max_run) {
    int best = 1;
    double least = 1e300;
    for (int r = 1; r <= std::min<int64_t>(depth, max_run); ++r) {
        const int64_t items = tiles * ((depth + r - 1) / r), slots = cus * kBlocksPerCu3;
        const double us = items <= cus ? 0.5 + 1.34 * r
                                       : (double)((items + slots - 1) / slots) * (3.9 + 1.71 * r);
        if (us <= least) {
            least = us;
            best = r;
        }
    }
    return best;
}

hipError_t launch_step_3d_f16(const StepArgs &a, const void *src, void *dst, const void *img,
                              int cdh, int cdw, int fz, int fy, int fx, hipStream_t stream) {
    Args3 b{};
    b.src = (const __half *)src;
    b.dst = (__half *)dst;
    b.img = (const __half *)img;
    b.seg = a.seg;
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
    b.tiles_x = (int)((a.ext.w + kTX - 1) / kTX);
    b.tiles_y = (int)((a.ext.h + kTY - 1) / kTY);
    b.cdh = cdh;
    b.cdw = cdw;
    b.fz = fz;
    b.fy = fy;
    b.fx = fx;
    b.level = a.level;
    b.step = a.step;
    b.batch = a.batch;
    const int64_t tiles = (int64_t)b.tiles_x * b.tiles_y;
    const int64_t cus = device_cus(), slots = cus * kBlocksPerCu3;
    b.zrun = step_3d_f16_run(tiles, a.ext.d, cus, a.ext.w % 8 == 0 ? kMaxRun : kMaxRun / 2);
    const int64_t items = tiles * ((a.ext.d + b.zrun - 1) / b.zrun);
    if (items == 0) return hipSuccess;
    if (items > INT32_MAX) return hipErrorInvalidValue;
    b.items = (int)items;
    const int grid = (int)std::min<int64_t>(items, slots);
    const bool up = img != nullptr, seg = a.seg != nullptr;
    if (up && seg) return hipErrorInvalidValue;
    if (a.n_in == 1)
        up ? launch3<1, true, false>(b, grid, stream)
           : seg ? launch3<1, false, true>(b, grid, stream) : launch3<1, false, false>(b, grid, stream);
    else
        up ? launch3<3, true, false>(b, grid, stream)
           : seg ? launch3<3, false, true>(b, grid, stream) : launch3<3, false, false>(b, grid, stream);
    return hipGetLastError();
}

}  // namespace octnca
