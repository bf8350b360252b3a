// Several NCA steps of a small 2D level in one launch (Sec. 3.1 step; the
// state between the steps stays on chip).
//
// A step of a small level is bound by latency, not by work: one launch, the
// weight prologue and one wave's rows cost about 6 us whatever the level's
// size, of which the arithmetic is a fraction.  Here a block of 8 waves owns
// a T x T tile: it loads the tile with a halo of k cells into LDS once and
// runs k steps there, on regions that shrink by one cell on each side per
// step (step s computes the tile grown by k - 1 - s cells), so no block needs
// another's results.  The price is the halo work that neighbouring blocks
// repeat; step_block_plan weighs it against the launches saved.  The fire
// mask is a function of (seed, level, step, cell) alone, so the copies of a
// halo cell agree.
//
// The state sits in LDS as fp32 channel-quad planes in two buffers (read one,
// write the other: one block barrier per step).  A work unit is 16 columns x
// 2 rows: lane (n, g) owns channel quad g of column n, reads 4 x 3 cells for
// the perception of its two cells, and runs the MLP of the two 16-cell groups
// (lane layout, operand policies and operation order of the row kernels, so
// the results are the same bits).  Columns are enumerated across row pairs,
// so that ragged regions leave no lanes idle but the last unit's.
#include <algorithm>
#include <type_traits>

#include "launch.h"
#include "step_common.h"

namespace octnca {

namespace {

constexpr int kBlockWaves = 8;
constexpr int kBlockThreads = 64 * kBlockWaves;
constexpr int kRegionMax = 34;      // tile + halo on both sides
constexpr int kBlockMaxSteps = 10;
constexpr int kQuadPlane = plane_stride(kRegionMax * kRegionMax);   // 16-byte words

// Plans count the CUs of a full MI355X, not the device's, so that the launch
// sequence is the same on every device.
constexpr int64_t kPlanCus = 256;
// Above these sizes one launch per step wins (one step at 724^2, fp32 then
// fp16: 17.6 against 20.8 us, 14.7 against 18.1; 1001^2: 31.6 against 31.1,
// 27.8 against 27.0), or, for the training tape, nothing larger was timed.
constexpr int64_t kBlockMaxCells = 600000, kTapeMaxCells = 400000, kBlockMaxSide = 400000;
constexpr double kTurnUs = 1.05, kTurnF16Us = 0.88, kTapeTurnUs = 1.5;

struct BlockArgs {
    const void *src;      // the level's state; the coarse state with an upsample; unused for a seed
    void *dst;            // state after the last step, or the tape (TAPE: state after step s at
                          // dst + s * tape_stride elements)
    const void *img;      // the level's image (upsample / seed)
    uint8_t *seg;         // readout of dst, or null
    const float *conv_w, *conv_b, *w1, *b1, *w2;
    uint64_t seed, threshold;
    int64_t tape_stride;
    int64_t src_stride, dst_stride, img_stride, seg_stride;   // elements between images
    int dh, dw, cdw, fy, fx;
    int tile, tiles_x, steps;
    uint32_t level, step, batch;
};

// How the first state of a launch is formed.
enum class BlockIn : int {
    State = 0,      // a state of this level
    Upsample = 1,   // the coarser level's state and this level's image
    Seed = 2,       // this level's image, zero hidden channels
};

template <typename T, int NIN, class Mlp, BlockIn IN, bool TAPE>
__global__ __launch_bounds__(kBlockThreads, 1) void nca_steps_block_2d(const BlockArgs A) {
    constexpr int C = Mlp::kChannels;
    using Ch = CellChunk<T, C>;
    constexpr int NQ = Ch::N;
    constexpr int kCellBytes = C * (int)sizeof(T);
    constexpr int kChunks = Ch::kUsed;
    constexpr int kCellsPerLoad = 64 / NQ;               // cells a wave's load covers
    constexpr int kMaxLoads =
        (kRegionMax * kRegionMax + kCellsPerLoad * kBlockWaves - 1) / (kCellsPerLoad * kBlockWaves);
    __shared__ float4 state[2][4 * kQuadPlane];
    __shared__ uint64_t fire[kBlockMaxSteps][kRegionMax];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15;
    const int g = lane >> 4;
    const int k = A.steps;
    const int image = blockIdx.y;
    const int ty = blockIdx.x / A.tiles_x;
    const int y0 = ty * A.tile, x0 = (blockIdx.x - ty * A.tiles_x) * A.tile;
    const int rw = A.tile + 2 * k;                       // region width and height, LDS row stride
    const int ry0 = y0 - k, rx0 = x0 - k;                // the region's first cell
    const T *src = (const T *)A.src + image * A.src_stride;
    const T *img = (const T *)A.img + image * A.img_stride;

    // 1. the region's cells, in registers until the weights are gathered
    const int rcells = rw * rw;
    const uint32_t rmagic = (65536u + rw - 1) / rw;      // e / rw for e < 65536 / rw (1927 > 34 * 34)
    const uint32_t cells = (uint32_t)A.dh * A.dw;
    uint4 v[kMaxLoads];
    {
        const Rsrc r = IN == BlockIn::Seed ? make_rsrc(A.conv_b, 0)
                       : IN == BlockIn::Upsample
                           ? make_rsrc(src, (uint32_t)(A.dh / A.fy) * A.cdw * kCellBytes)
                           : make_rsrc(src, cells * kCellBytes);
        const int chunk = lane / kCellsPerLoad;
#pragma unroll
        for (int j = 0; j < kMaxLoads; ++j) {
            const int e = (j * kBlockWaves + wave) * kCellsPerLoad + lane % kCellsPerLoad;
            const int ly = (int)(((uint32_t)e * rmagic) >> 16);
            const int y = ry0 + ly, x = rx0 + e - ly * rw;
            const bool ok = e < rcells && chunk < kChunks && y >= 0 && y < A.dh && x >= 0 && x < A.dw;
            uint32_t cell;
            if constexpr (IN == BlockIn::Upsample)
                // exact for y, x < 2^19: (y + 1/2) / f stays 1/16 away from the next integer
                cell = (uint32_t)((int)(((float)y + 0.5f) * (1.f / A.fy)) * A.cdw +
                                  (int)(((float)x + 0.5f) * (1.f / A.fx)));
            else
                cell = (uint32_t)(y * A.dw + x);
            v[j] = Ch::load(r, ok ? cell * kCellBytes + (uint32_t)(chunk * Ch::kBytes) : kOut);
        }
    }
    // image values of the region's input channels (one cell per thread and turn)
    constexpr int kImgLoads = (kRegionMax * kRegionMax + kBlockThreads - 1) / kBlockThreads;
    float im[IN == BlockIn::State ? 1 : kImgLoads][NIN];
    if constexpr (IN != BlockIn::State) {
        const Rsrc r = make_rsrc(img, cells * NIN * (uint32_t)sizeof(T));
#pragma unroll
        for (int j = 0; j < kImgLoads; ++j) {
            const int e = j * kBlockThreads + (int)threadIdx.x;
            const int ly = (int)(((uint32_t)e * rmagic) >> 16);
            const int y = ry0 + ly, x = rx0 + e - ly * rw;
            const bool ok = e < rcells && y >= 0 && y < A.dh && x >= 0 && x < A.dw;
#pragma unroll
            for (int c = 0; c < NIN; ++c) {
                const uint32_t off =
                    ok ? (uint32_t)((y * A.dw + x) * NIN + c) * (uint32_t)sizeof(T) : kOut;
                if constexpr (sizeof(T) == 4)
                    im[j][c] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
                else
                    im[j][c] = __half2float(__ushort_as_half(
                        (unsigned short)__builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0)));
            }
        }
    }

    // 2. weights, one copy per block: gathered by every wave from memory they
    // cost 2.3 us of a 7.9 us launch (16 cache lines per load instruction, 8
    // waves), so the block loads them once, contiguous, and the waves gather
    // from LDS.  Rows are padded to an odd number of 16-byte words there (no
    // bank conflicts between the 16 rows a gather touches).
    constexpr int H = Mlp::kHidden;
    constexpr int kLd1 = 2 * C + 4, kLd2 = H + 4;
    constexpr int kW2At = H * kLd1, kB1At = kW2At + C * kLd2, kTapAt = kB1At + H,
                  kCbAt = kTapAt + 9 * C;
    static_assert((kCbAt + C) * 4 <= (int)sizeof(state[1]), "the copy fits the second buffer");
    float *const wcopy = reinterpret_cast<float *>(state[1]);
    constexpr int kW1Loads = (H * 2 * C + kBlockThreads - 1) / kBlockThreads;
    constexpr int kW2Loads = (C * H + kBlockThreads - 1) / kBlockThreads;
    static_assert(H + 10 * C <= kBlockThreads, "one load for the biases and taps");
    float wv[kW1Loads + kW2Loads + 1];
    {
        const int t = threadIdx.x;
#pragma unroll
        for (int j = 0; j < kW1Loads; ++j) wv[j] = A.w1[min(t + j * kBlockThreads, H * 2 * C - 1)];
#pragma unroll
        for (int j = 0; j < kW2Loads; ++j)
            wv[kW1Loads + j] = A.w2[min(t + j * kBlockThreads, C * H - 1)];
        const float *rest = t < H            ? A.b1 + t
                            : t < H + 9 * C  ? A.conv_w + (t - H)
                                             : A.conv_b + min(t - H - 9 * C, C - 1);
        wv[kW1Loads + kW2Loads] = *rest;
    }

    // 3. fire bits of all steps, on the first step's region (the widest):
    // bit (idx0 & 7) + x - xa of a row's word is the draw of cell x, idx0 the
    // canonical index of the row's first cell
    const int e1 = k - 1;
    const int ya1 = max(0, y0 - e1), yb1 = min(A.dh, y0 + A.tile + e1);
    const int xa1 = max(0, x0 - e1), xb1 = min(A.dw, x0 + A.tile + e1);
    {
        const int rows = yb1 - ya1;
        const int nb = (xb1 - xa1 + 14) >> 3;            // 8-cell blocks a row can touch
        const int per_step = rows * nb;
        for (int i = threadIdx.x; i < k * per_step; i += kBlockThreads) {
            const int s = i / per_step;
            const int rb = i - s * per_step;
            const int row = rb / nb, b = rb - row * nb;
            const uint64_t b0 = ((uint64_t)(ya1 + row) * A.dw + xa1) >> 3;
            const Philox4x64Out p = philox4x64_10(b0 + b, A.step + s, A.level, A.batch + image,
                                                  A.seed, 0);
            uint32_t bits = 0;
#pragma unroll
            for (int c = 0; c < 8; ++c)
                bits |= ((uint64_t)draw_of(p, (uint32_t)c) < A.threshold ? 1u : 0u) << c;
            reinterpret_cast<uint8_t *>(&fire[s][row])[b] = (uint8_t)bits;
        }
    }

    // 4. the region and the weights into LDS
    {
        const int chunk = lane / kCellsPerLoad;
#pragma unroll
        for (int j = 0; j < kMaxLoads; ++j) {
            const int e = (j * kBlockWaves + wave) * kCellsPerLoad + lane % kCellsPerLoad;
            if (e < rcells) Ch::put(state[0], kQuadPlane, chunk, e, v[j]);
        }
        const int t = threadIdx.x;
#pragma unroll
        for (int j = 0; j < kW1Loads; ++j) {
            const int i = min(t + j * kBlockThreads, H * 2 * C - 1);
            wcopy[i / (2 * C) * kLd1 + i % (2 * C)] = wv[j];
        }
#pragma unroll
        for (int j = 0; j < kW2Loads; ++j) {
            const int i = min(t + j * kBlockThreads, C * H - 1);
            wcopy[kW2At + i / H * kLd2 + i % H] = wv[kW1Loads + j];
        }
        if (t < H + 10 * C) wcopy[kB1At + t] = wv[kW1Loads + kW2Loads];
    }
    __syncthreads();
    Mlp mlp;
    mlp.load(wcopy, wcopy + kB1At, wcopy + kW2At, n, g, NIN, kLd1, kLd2);
    float tap[9][4], cb[4];
    {
        const bool g_ok = g < C / 4;
        const int gc = g_ok ? g : 0;
        constexpr float ps = Mlp::kPerceptionScale;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                const float w = wcopy[kTapAt + (4 * gc + q) * 9 + t];
                tap[t][q] = g_ok ? ps * w : 0.f;
            }
            const float b = wcopy[kCbAt + 4 * gc + q];
            cb[q] = g_ok ? ps * b : 0.f;
        }
    }
    // the gathers complete here, not inside the step loop
    mlp.pin_all();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int t = 0; t < 9; ++t) pin(tap[t][q]);
        pin(cb[q]);
    }
    // image values go over quad 0, which other waves wrote
    if constexpr (IN != BlockIn::State) {
#pragma unroll
        for (int j = 0; j < kImgLoads; ++j) {
            const int e = j * kBlockThreads + (int)threadIdx.x;
            if (e < rcells)
#pragma unroll
                for (int c = 0; c < NIN; ++c) reinterpret_cast<float *>(&state[0][e])[c] = im[j][c];
        }
    }
    __syncthreads();
    // cells outside the grid are zero in both buffers: the zero padding
    if (ry0 < 0 || rx0 < 0 || ry0 + rw > A.dh || rx0 + rw > A.dw) {
        for (int i = threadIdx.x; i < 4 * rcells; i += kBlockThreads) {
            const int q = i / rcells;
            state[1][q * kQuadPlane + i - q * rcells] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        __syncthreads();
    }

    // 5. the steps
    const uint32_t out_bytes = cells * kCellBytes;
    T *dst = (T *)A.dst + image * A.dst_stride;
    for (int s = 0; s < k; ++s) {
        const int e = k - 1 - s;
        const int ya = max(0, y0 - e), yb = min(A.dh, y0 + A.tile + e);
        const int xa = max(0, x0 - e), xb = min(A.dw, x0 + A.tile + e);
        const int w = xb - xa, h = yb - ya;
        const int total = ((h + 1) >> 1) * w;            // columns of row pairs
        const uint32_t magic = (65536u + w - 1) / w;
        const float4 *in = state[s & 1] + g * kQuadPlane;
        float4 *out = state[(s + 1) & 1] + g * kQuadPlane;
        const bool last = s + 1 == k;
        const Rsrc wr = make_rsrc(TAPE ? dst + s * A.tape_stride : dst,
                                  TAPE || last ? out_bytes : 0u);
        for (int u = wave * 16; u < total; u += kBlockWaves * 16) {
            const uint32_t col = (uint32_t)min(u + n, total - 1);
            const bool in_unit = u + n < total;
            const uint32_t pair = __umul24(col, magic) >> 16;
            const int x = xa + (int)(col - __umul24(pair, (uint32_t)w));
            const int y = ya + 2 * (int)pair;
            const bool two = 2 * (int)pair + 1 < h;
            const int base = __mul24(y - ry0, rw) + x - rx0;
            // the lower neighbour row of the second cell; its own row again
            // where the region ends (that cell is not kept then)
            const int row3 = base + (two ? 2 * rw : rw);
            // All LDS reads of the unit are issued before the first is used:
            // a small level has one unit per wave and step, and its time is
            // these reads' and the two MLPs' latency.
            float4 c[4][3];
            uint64_t bits[2];
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int dx = 0; dx < 3; ++dx)
                    c[r][dx] = in[(r < 3 ? base + (r - 1) * rw : row3) + dx - 1];
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int yr = min(y + r, yb - 1);
                const int sh = (int)((__umul24((uint32_t)yr, (uint32_t)A.dw & 7u) + xa1) & 7u) + x - xa1;
                bits[r] = fire[s][yr - ya1] >> sh;
            }
            __builtin_amdgcn_sched_barrier(0);
            float f[2][8];
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const float own[4] = {c[r + 1][1].x, c[r + 1][1].y, c[r + 1][1].z, c[r + 1][1].w};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    f[r][q] = own[q];
                    f[r][4 + q] = cb[q];
                }
#pragma unroll
                for (int t = 0; t < 9; ++t) {
                    const float4 v = c[r + t / 3][t % 3];
                    f[r][4] = fmaf(tap[t][0], v.x, f[r][4]);
                    f[r][5] = fmaf(tap[t][1], v.y, f[r][5]);
                    f[r][6] = fmaf(tap[t][2], v.z, f[r][6]);
                    f[r][7] = fmaf(tap[t][3], v.w, f[r][7]);
                }
            }
            v4f acc[2][4], up[2];
            mlp.layer1(f[0], acc[0]);
            mlp.layer1(f[1], acc[1]);
            up[0] = mlp.layer2(acc[0]);
            up[1] = mlp.layer2(acc[1]);
            float4 o[2];
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const float m = (float)((uint32_t)bits[r] & 1u);
                o[r] = make_float4(
                    gated<Mlp>(m, up[r][0], f[r][0]), gated<Mlp>(m, up[r][1], f[r][1]),
                    gated<Mlp>(m, up[r][2], f[r][2]), gated<Mlp>(m, up[r][3], f[r][3]));
                if constexpr (sizeof(T) == 2) {          // stored precision between the steps
                    o[r].x = __half2float(__float2half_rn(o[r].x));
                    o[r].y = __half2float(__float2half_rn(o[r].y));
                    o[r].z = __half2float(__float2half_rn(o[r].z));
                    o[r].w = __half2float(__float2half_rn(o[r].w));
                }
            }
            if (!last && in_unit) {
                out[base] = o[0];
                if (two) out[base + rw] = o[1];
            }
            if (TAPE || last) {
                const bool own_x = in_unit && g < C / 4 && x >= x0 && x < x0 + A.tile;
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const bool own = own_x && (r == 0 || two) && y + r >= y0 && y + r < y0 + A.tile;
                    const uint32_t cell = (uint32_t)((y + r) * A.dw + x);
                    store_quad(dst, wr, own ? cell * kCellBytes : kOut, g,
                               v4f{o[r].x, o[r].y, o[r].z, o[r].w});
                    if (last && A.seg != nullptr) {
                        constexpr int q = (C - 1) / 4;
                        static_assert((C - 1) % 4 == 3, "the readout channels share a quad");
                        if (own && g == q)
                            A.seg[image * A.seg_stride + cell] = o[r].w > o[r].z ? 1 : 0;
                    }
                }
            }
        }
        if (!last) __syncthreads();
    }
}

template <typename T, class Mlp, BlockIn IN, bool TAPE>
void launch_block_nin(const BlockArgs &b, int n_in, dim3 grid, hipStream_t stream) {
    if (n_in == 1)
        nca_steps_block_2d<T, 1, Mlp, IN, TAPE><<<grid, kBlockThreads, 0, stream>>>(b);
    else
        nca_steps_block_2d<T, 3, Mlp, IN, TAPE><<<grid, kBlockThreads, 0, stream>>>(b);
}

template <typename T, class Mlp>
void launch_block_in(const BlockArgs &b, int n_in, BlockIn in, dim3 grid, hipStream_t stream) {
    switch (in) {
        case BlockIn::State:
            return launch_block_nin<T, Mlp, BlockIn::State, false>(b, n_in, grid, stream);
        case BlockIn::Upsample:
            return launch_block_nin<T, Mlp, BlockIn::Upsample, false>(b, n_in, grid, stream);
        case BlockIn::Seed:
            return launch_block_nin<T, Mlp, BlockIn::Seed, false>(b, n_in, grid, stream);
    }
}

bool is_size(const StepArgs &a, int c, int h) { return a.channels == c && a.hidden == h; }

}  // namespace

namespace {

// Time model of the launches that run `steps` steps on T x T tiles, at most k
// per launch, in us: 2.4 for a launch, and for each round of blocks (one block
// per CU: its LDS) 2.8 until its first step (loads, weights, fire bits) and
// one turn of 8 units per kTurnUs (fp16 operands: kTurnF16Us).  Measured, C = 16 fp32: 9.4 / 9.9 / 10.6 /
// 13.4 / 20.8 us for 5 steps of 16^2 (T 4), 16^2 (8), 128^2 (8), 4 of 256^2
// (16), 5 of 320^2 (20); the model gives 10.5 / 10.5 / 10.5 / 12.6 / 19.9.
constexpr double kLaunchUs = 2.4, kBlockUs = 2.8;

double block_cost(int64_t h, int64_t w, int images, int steps, int tile, int launches,
                  double turn_us) {
    const int64_t blocks = (h + tile - 1) / tile * ((w + tile - 1) / tile) * images;
    const double rounds = (double)((blocks + kPlanCus - 1) / kPlanCus);
    auto one = [&](int k) {
        int64_t turns = 0;
        for (int e = 0; e < k; ++e) {
            const int64_t rh = std::min<int64_t>(h, tile + 2 * e);
            const int64_t cols = (rh + 1) / 2 * std::min<int64_t>(w, tile + 2 * e);
            turns += (cols + 16 * kBlockWaves - 1) / (16 * kBlockWaves);
        }
        return kLaunchUs + rounds * (kBlockUs + turn_us * (double)turns);
    };
    const int more = steps % launches;   // launches with one step more
    return (more ? more * one(steps / launches + 1) : 0.0) +
           (launches - more) * one(steps / launches);
}

}  // namespace

bool step_block_plan(const StepArgs &a, bool tape, int steps, int images, StepBlockPlan *plan,
                     bool same_parity) {
    if (a.ndim != 2 || steps < 1) return false;
    if (tape) {
        if (a.dtype != Dtype::F32 || !is_size(a, 16, 64)) return false;
    } else {
        if (a.kc.valu || !a.kc.pairs || a.kc.layout != Layout2d::Auto) return false;
        const bool mlp_ok = a.kc.mlp == MfmaMlp::Default ||
                            a.kc.mlp == (a.dtype == Dtype::F32 ? MfmaMlp::F16S : MfmaMlp::F16);
        if (!mlp_ok) return false;
        if (!is_size(a, 16, 64) && !is_size(a, 12, 48)) return false;
    }
    // (the kernel's exact divisions need h, w < 2^19, its offsets 32 bits)
    const int64_t h = a.ext.h, w = a.ext.w;
    const int64_t max_cells = tape ? kTapeMaxCells : kBlockMaxCells;
    if (h > kBlockMaxSide || w > kBlockMaxSide || h * w > max_cells) return false;
    const double turn_us = tape ? kTapeTurnUs : a.dtype == Dtype::F16 ? kTurnF16Us : kTurnUs;
    // One launch per step on the row kernel, measured: 5.0 us up to 128^2
    // cells, 6.8 at 256^2, 8.8 at 320^2, 11.3 at 512^2, 27.7 at 1024^2; where
    // rows do not start on 8-cell boundaries 14.3 at 600^2, 20.8 at 724^2
    // (the training forward about 1 us more).  The images of a batch would run
    // one after another there.
    double best = (double)steps * images *
                  ((tape ? 5.5 : 4.5) + (double)(h * w) / (w % 8 == 0 ? 45000.0 : 33000.0));
    bool use = false;
    for (int tile : {4, 6, 8, 10, 12, 14, 16, 18, 20, 22, 24, 28}) {
        if (tile > 4 && tile / 2 >= std::max(h, w)) break;
        int last = 0;
        for (int k = std::min({(kRegionMax - tile) / 2, kBlockMaxSteps, steps}); k >= 1; --k) {
            int launches = (steps + k - 1) / k;
            if (same_parity) launches += (launches ^ steps) & 1;
            if (launches == last) continue;
            last = launches;
            const double c = block_cost(h, w, images, steps, tile, launches, turn_us);
            if (c < best) {
                best = c;
                plan->tile = tile;
                plan->launches = launches;
                use = true;
            }
        }
    }
    plan->us = best;
    return use;
}

hipError_t launch_step_block(const StepArgs &a, bool tape, int tile, int steps, const void *src,
                             void *dst, StepBlockInput in, hipStream_t stream) {
    if (steps < 1 || steps > kBlockMaxSteps || tile < 1 || tile + 2 * steps > kRegionMax)
        return hipErrorInvalidValue;
    BlockArgs b{};
    b.src = src;
    b.dst = dst;
    b.img = in.img;
    b.seg = a.seg;
    b.conv_w = a.w.conv_w;
    b.conv_b = a.w.conv_b;
    b.w1 = a.w.w1;
    b.b1 = a.w.b1;
    b.w2 = a.w.w2;
    b.seed = a.seed;
    b.threshold = a.threshold;
    b.tape_stride = a.ext.cells() * a.channels;
    b.src_stride = in.src_stride;
    b.dst_stride = in.dst_stride;
    b.img_stride = in.img_stride;
    b.seg_stride = a.ext.cells();
    b.dh = (int)a.ext.h;
    b.dw = (int)a.ext.w;
    b.cdw = in.coarse_w;
    b.fy = in.fy;
    b.fx = in.fx;
    b.tile = tile;
    b.tiles_x = (int)((a.ext.w + tile - 1) / tile);
    b.steps = steps;
    b.level = a.level;
    b.step = a.step;
    b.batch = a.batch;
    const int64_t blocks = (int64_t)b.tiles_x * ((a.ext.h + tile - 1) / tile);
    if (blocks > INT32_MAX || in.images < 1 || in.images > 65535) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks, (unsigned)in.images);
    const BlockIn how = in.img == nullptr ? BlockIn::State
                        : src == nullptr  ? BlockIn::Seed
                                          : BlockIn::Upsample;
    if (tape) {
        if (how != BlockIn::State) return hipErrorInvalidValue;
        launch_block_nin<float, MlpBf16x3, BlockIn::State, true>(b, a.n_in, grid, stream);
    } else if (a.dtype == Dtype::F16 && is_size(a, 12, 48)) {
        launch_block_in<__half, MlpF16M<12, 48>>(b, a.n_in, how, grid, stream);
    } else if (a.dtype == Dtype::F16) {
        launch_block_in<__half, MlpF16>(b, a.n_in, how, grid, stream);
    } else if (is_size(a, 12, 48)) {
        launch_block_in<float, MlpF16SM<12, 48>>(b, a.n_in, how, grid, stream);
    } else {
        launch_block_in<float, MlpF32State>(b, a.n_in, how, grid, stream);
    }
    return hipGetLastError();
}

}  // namespace octnca
