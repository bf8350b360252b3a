// Fused NCA step on the matrix cores (Sec. 3.1; supplement S3, Listing 1).
//
// The per-cell MLP 2C -> H -> C is a dense contraction over a batch of
// cells, so it runs on MFMA; perception, ReLU, the fire gate and the
// residual stay on the VALU.
//
// Lane mapping (wave64, one "group" = 16 cells handled by one MFMA chain):
//   lane l -> cell n = l % 16 of the group, channel quad g = l / 16, i.e. the
//   lane owns channels 4g .. 4g+3 of its cell.
//   * it computes the perception of those 4 channels (depthwise taps read
//     from an LDS tile with a one-cell halo, zero padding outside the grid);
//   * layer 1, H[j][n] = b1[j] + sum_k W1[j][k] F[n][k], runs as
//     v_mfma_f32_16x16x4_f32 with A = W1 tile (16 hidden units x 4
//     features), B = features (4 x 16 cells).  The B operand of lane l is
//     feature row k = l / 16 of its cell, so feature chunk kc is taken as
//     state channel 4g + kc (kc < 4) or perception channel 4g + kc - 4;
//     W1's columns are gathered in the same order.  4 hidden tiles x 8
//     feature chunks = 32 MFMAs per group;
//   * the accumulator of hidden tile jt leaves hidden unit jt*16 + 4g + i of
//     cell n in register i of lane l, which is exactly the B operand layout
//     of the second layer with K index g; so after ReLU the registers feed
//     layer 2 (U[c][n] = sum_j W2[c][j] H[j][n]) directly, 16 MFMAs, with
//     W2's columns gathered to match.  No hidden value leaves the registers;
//   * layer 2's accumulator holds channels 4g .. 4g+3 of cell n in lane l:
//     the channels whose state the lane already holds, so the residual
//     update and the 16-byte store need no data exchange.
// Fire bits: each lane evaluates Philox4x64-10 for one block of 8 cells of
// the rows its wave owns (covering several tiles or planes ahead), the bits
// are spread with eight ballots and every lane picks its cell's bit.
//
// 2D: a persistent grid loops over 16 x 32 tiles; the 18 x 34 halo tile is
// staged in LDS as fp32 in four channel-quad planes (conflict-free 16-byte
// reads).  3D: a block owns an 8 x 32 column of the (y, x) plane and a run
// of z planes, keeping three halo planes in an LDS ring (each plane is read
// from HBM once per run).
#include <atomic>
#include <algorithm>
#include <type_traits>

#include "launch.h"
#include "step_common.h"

namespace octnca {

namespace {

constexpr int kThreads = 256;   // 4 waves

// Per-lane view of one evaluation: `mine` is the ballot of the lane's cells
// when rows are 8-aligned.
struct FireBits {
    FireBallots f;
    uint64_t mine;
    bool aligned;
    int opr;

    // Bit of cell idx in row slot `slot` whose first block is row_b0.
    __device__ __forceinline__ bool bit(int slot, uint64_t idx, uint64_t row_b0) const {
        const int o = (int)((idx >> 3) - row_b0);
        const uint64_t w = aligned ? mine : select_ballot(f, (uint32_t)idx & 7u);
        return (w >> (slot * opr + o)) & 1;
    }

};

// ---------------------------------------------------------------------------
// Halo tiles: HY rows of 34 cells (a 32-cell-wide interior plus one halo cell
// on each side) of one z plane.  In LDS they are kept as fp32 in four
// channel-quad planes, so that the 16 lanes of a quad read 16 consecutive
// 16-byte words (no bank conflicts); the plane stride is 2 mod 8 (16-byte
// words, see plane_stride).
// Loads are whole 16-byte chunks: a "body" load moves the 64 chunks of a row
// segment (16 cells in fp32, 32 in fp16) from one wave-uniform address, a
// "side" load moves the left and right halo cells of several rows.  The loads are spread over the 4 waves
// and go through registers: the next tile's loads are issued before the
// current tile is computed and written to LDS after it (software
// pipelining), so HBM latency overlaps the compute.
// ---------------------------------------------------------------------------
constexpr int kTileW = 32;
constexpr int kHaloW = kTileW + 2;

// C: channels of a cell; a cell fills kChunks of the NQ 16-byte chunks, the
// loads of the others (channel quad 3 when C = 12) take the out-of-range
// offset and read as zero.
template <typename T, int HY, int C = kC>
struct RowLoader {
    using Ch = CellChunk<T, C>;
    static constexpr int NQ = Ch::N;
    static constexpr int kCellBytes = C * (int)sizeof(T);
    static constexpr int kChunks = Ch::kUsed;
    static constexpr int kCellsPerBody = 64 / NQ;            // cells per body load
    static constexpr int kBodyPerRow = kTileW / kCellsPerBody;
    static constexpr int kRowsPerSide = 64 / (2 * NQ);       // rows per side load
    static constexpr int kBody = HY * kBodyPerRow;
    static constexpr int kSide = (HY + kRowsPerSide - 1) / kRowsPerSide;
    static constexpr int kBodySlots = (kBody + 3) / 4;       // body loads per wave (max)
    static_assert(kSide <= 4, "one side load per wave at most");
    static constexpr int PS = plane_stride(HY * kHaloW);
    // Body load J (0 <= J < kBody) is slot J / 4 of wave J % 4: every wave
    // runs the same instruction sequence.  Side load s is done by wave 3 - s,
    // in one extra slot.
    uint4 v[kBodySlots + 1];

    // A body load moves the kCellsPerBody cells x NQ chunks of a row segment.
    // Lane i takes chunk i / kCellsPerBody of cell i % kCellsPerBody: the
    // wave still reads one contiguous 1 KB, and each group of consecutive
    // lanes writes consecutive 16-byte words of one LDS plane (no bank
    // conflicts on the commit).
    __device__ static __forceinline__ int body_cell(int lane) { return lane % kCellsPerBody; }
    __device__ static __forceinline__ int body_chunk(int lane) { return lane / kCellsPerBody; }

    // Per-lane byte offsets of a tile's loads within its rows (kOut for
    // unused slots and for cells left of x = 0, above y = 0 or right of the
    // grid; rows below the grid fall outside the descriptor).  They depend on
    // the tile only, so a plane loop computes them once per work item and
    // issue_at() changes only the descriptor from plane to plane.
    struct Offsets {
        uint32_t o[kBodySlots + 1];
    };
    __device__ __forceinline__ static Offsets offsets(int dw, int y0, int x0) {
        const int lane = threadIdx.x & 63;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int gy0 = y0 - 1;
        const int base_row = gy0 > 0 ? gy0 : 0;
        const uint32_t row_bytes = (uint32_t)dw * kCellBytes;
        const int cell = body_cell(lane);
        const uint32_t lane_off = (uint32_t)(cell * kCellBytes + body_chunk(lane) * Ch::kBytes);
        Offsets r;
#pragma unroll
        for (int k = 0; k < kBodySlots; ++k) {
            const int J = wave + 4 * k;                       // wave-uniform
            const int gy = gy0 + J / kBodyPerRow;
            const int cx0 = x0 + (J % kBodyPerRow) * kCellsPerBody;
            const bool ok = J < kBody && gy >= 0 && cx0 + cell < dw && body_chunk(lane) < kChunks;
            const uint32_t off = (uint32_t)(gy - base_row) * row_bytes +
                                 (uint32_t)cx0 * kCellBytes + lane_off;
            r.o[k] = ok ? off : kOut;
        }
        const int s = 3 - wave;
        const int row = s * kRowsPerSide + lane / (2 * NQ);
        const int gy = gy0 + row;
        const int gx = ((lane / NQ) & 1) ? x0 + kTileW : x0 - 1;
        const bool ok =
            s < kSide && row < HY && gy >= 0 && gx >= 0 && gx < dw && lane % NQ < kChunks;
        const uint32_t off = (uint32_t)(gy - base_row) * row_bytes + (uint32_t)gx * kCellBytes +
                             (uint32_t)(lane % NQ) * Ch::kBytes;
        r.o[kBodySlots] = ok ? off : kOut;
        return r;
    }

    // Tile whose interior starts at (y0, x0) in plane z (lane offsets `of`
    // from offsets()); cells outside the grid (or z outside [0, dd)) read as
    // zero.  The grid must satisfy HY * dw * kCellBytes < 2^32 (checked by
    // the launcher).  With active = false nothing is read (the descriptor is
    // empty) and the registers are zero: the next-tile prefetch is issued
    // unconditionally.
    __device__ __forceinline__ void issue_at(const T *__restrict__ src, const Offsets &of, int z,
                                             int dd, int dh, int dw, int y0, bool active = true) {
        const int gy0 = y0 - 1;
        const int base_row = gy0 > 0 ? gy0 : 0;
        const int rows =
            (active && z >= 0 && z < dd) ? max(0, min(gy0 + HY, dh) - base_row) : 0;
        const uint32_t row_bytes = (uint32_t)dw * kCellBytes;
        const Rsrc r = make_rsrc(src + ((int64_t)max(z, 0) * dh + base_row) * dw * C,
                                 (uint32_t)rows * row_bytes);
#pragma unroll
        for (int k = 0; k <= kBodySlots; ++k) {
            v[k] = Ch::load(r, of.o[k]);
        }
    }
    __device__ __forceinline__ void issue(const T *__restrict__ src, int z, int dd, int dh, int dw,
                                          int y0, int x0, bool active = true) {
        issue_at(src, offsets(dw, y0, x0), z, dd, dh, dw, y0, active);
    }

    __device__ __forceinline__ static void put(float4 *planes, int q, int cell, const uint4 &c) {
        Ch::put(planes, PS, q, cell, c);
    }

    // LDS slot that is never read (plane padding): target of the writes of
    // unused load slots, so the commit has no branches either.
    static constexpr int kDummyCell = HY * kHaloW;
    static_assert(kDummyCell < PS, "plane padding holds the dummy slot");

    __device__ __forceinline__ void commit(float4 *planes) const {
        const int lane = threadIdx.x & 63;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int cell = body_cell(lane), chunk = body_chunk(lane);
#pragma unroll
        for (int k = 0; k < kBodySlots; ++k) {
            const int J = wave + 4 * k;
            const int slot =
                (J / kBodyPerRow) * kHaloW + 1 + (J % kBodyPerRow) * kCellsPerBody + cell;
            put(planes, chunk, J < kBody ? slot : kDummyCell, v[k]);
        }
        const int s = 3 - wave;
        const int row = s * kRowsPerSide + lane / (2 * NQ);
        const int slot = row * kHaloW + (((lane / NQ) & 1) ? kHaloW - 1 : 0);
        put(planes, lane % NQ, (s < kSide && row < HY) ? slot : kDummyCell, v[kBodySlots]);
    }
};

// Perception of channels 4g..4g+3 of the cell at LDS slot `centre`: the
// cell's own state in f[0..4), bias + taps in f[4..8).  `pl` points at the
// lane's channel-quad plane(s); tapw holds the conv weights as [tap][quad].
__device__ __forceinline__ void perceive_2d(const float4 *pl, const float4 (*tapw)[4], int g,
                                            int centre, const float cb[4], float f[8]) {
    const float4 sv = pl[centre];
    f[0] = sv.x; f[1] = sv.y; f[2] = sv.z; f[3] = sv.w;
    float p[4] = {cb[0], cb[1], cb[2], cb[3]};
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        const float4 v = pl[centre + (t / 3 - 1) * kHaloW + (t % 3 - 1)];
        const float4 w = tapw[t][g];
        p[0] = fmaf(w.x, v.x, p[0]);
        p[1] = fmaf(w.y, v.y, p[1]);
        p[2] = fmaf(w.z, v.z, p[2]);
        p[3] = fmaf(w.w, v.w, p[3]);
    }
    f[4] = p[0]; f[5] = p[1]; f[6] = p[2]; f[7] = p[3];
}

// ---------------------------------------------------------------------------
// 2D: persistent blocks loop over 16 x 32 tiles (tile index row-major); wave
// w computes rows 4w .. 4w+3 of the tile, 8 groups of 16 cells.
// ---------------------------------------------------------------------------
constexpr int k2TY = 16;
constexpr int k2BlocksPerCu = 2;   // 2 waves per SIMD: <= 256 VGPRs

template <typename T, int NIN, class Mlp>
__global__ __launch_bounds__(kThreads, k2BlocksPerCu) void nca_step_mfma_2d(
    const T *__restrict__ src, T *__restrict__ dst, int dh, int dw, int tiles_x, int tiles,
    const float *__restrict__ conv_w, const float *__restrict__ conv_b,
    const float *__restrict__ w1, const float *__restrict__ b1, const float *__restrict__ w2,
    uint32_t level, uint32_t step, uint32_t batch, uint64_t seed, uint64_t threshold) {
    static_assert(Mlp::kChannels == kC && Mlp::kHidden == kH, "built for C = 16, H = 64");
    using Loader = RowLoader<T, k2TY + 2>;
    __shared__ float4 planes[4 * Loader::PS];
    __shared__ float4 tapw[9][4];       // [tap][quad] conv weights of channels 4q..4q+3

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15;
    const int g = lane >> 4;

    {
        const int i = (int)threadIdx.x % (9 * 4);
        const int t = i / 4, q = i % 4;
        constexpr float ps = Mlp::kPerceptionScale;
        const float4 tw = make_float4(ps * conv_w[(4 * q + 0) * 9 + t], ps * conv_w[(4 * q + 1) * 9 + t],
                                      ps * conv_w[(4 * q + 2) * 9 + t], ps * conv_w[(4 * q + 3) * 9 + t]);
        tapw[t][q] = tw;   // threads >= 36 rewrite an entry (same value): no branch
    }
    Mlp mlp;
    mlp.load(w1, b1, w2, n, g, NIN);
    float cb[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) cb[k] = Mlp::kPerceptionScale * conv_b[4 * g + k];
    // all weight loads done before the tile loop (keeps the compiler's
    // vector-memory counting exact inside it)
    mlp.pin_all();
#pragma unroll
    for (int k = 0; k < 4; ++k) pin(cb[k]);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    // Fire evaluations: a tile's 4 rows per wave take 4 * opr lanes, so one
    // evaluation serves 64 / (4 opr) consecutive tiles of this block (4 when
    // rows are 8-aligned, else 2).
    FireBits fire;
    fire.aligned = (dw & 7) == 0;
    fire.opr = fire.aligned ? 4 : 8;
    const int lg_opr = fire.aligned ? 2 : 3;
    const int tiles_per_eval = 64 / (4 * fire.opr);
    const int stride = (int)gridDim.x;
    constexpr int kCellBytes = Loader::kCellBytes;
    const uint32_t row_bytes = (uint32_t)dw * kCellBytes;

    // The tile's halo is in LDS when an iteration starts: the first tile is
    // staged here, each later one is loaded during the previous iteration's
    // compute and written to LDS at its end (so every wait for those loads
    // sees the same history of memory operations).
    Loader ld;
    int tile = blockIdx.x;
    if (tile < tiles) {
        const int ty = tile / tiles_x;
        ld.issue(src, 0, 1, dh, dw, ty * k2TY, (tile - ty * tiles_x) * kTileW);
        ld.commit(planes);
    }
    for (int iter = 0; tile < tiles; tile += stride, ++iter) {
        const int ty = tile / tiles_x;
        const int y0 = ty * k2TY, x0 = (tile - ty * tiles_x) * kTileW;
        const int phase = iter & (tiles_per_eval - 1);
        if (phase == 0) {
            // lane -> (tile offset, row r of the wave's 4, block o of the row)
            const int tt = lane >> (lg_opr + 2);
            int t2 = tile + tt * stride;
            t2 = t2 < tiles ? t2 : tile;
            const int ty2 = t2 / tiles_x;
            const uint64_t row = (uint64_t)(ty2 * k2TY + 4 * wave + ((lane >> lg_opr) & 3));
            const uint64_t b0 = (row * dw + (uint64_t)(t2 - ty2 * tiles_x) * kTileW) >> 3;
            fire.f = fire_ballots(b0 + (lane & (fire.opr - 1)), step, level, batch, seed, threshold);
            fire.mine = select_ballot(fire.f, (uint32_t)n & 7u);
        }
        const int slot0 = phase * 4;
        __syncthreads();
        {
            const int next = tile + stride;
            const bool more = next < tiles;
            const int nt = more ? next : tile;
            const int nty = nt / tiles_x;
            ld.issue(src, 0, 1, dh, dw, nty * k2TY, (nt - nty * tiles_x) * kTileW, more);
        }

        // stores of this tile: rows y0 .. y0 + k2TY - 1 (clipped to the grid)
        const Rsrc wr = make_rsrc(dst + (int64_t)y0 * dw * kC,
                                  (uint32_t)min(k2TY, dh - y0) * row_bytes);
        // groups are software-pipelined: group grp + 1's perception is issued
        // while group grp's first-layer MFMAs run
        const float4 *pl = planes + g * Loader::PS;
        auto centre_of = [&](int grp) {
            return (4 * wave + (grp >> 1) + 1) * kHaloW + (grp & 1) * 16 + n + 1;
        };
        float f[8];
        perceive_2d(pl, tapw, g, centre_of(0), cb, f);
        // fully unrolled: with a counted sequence of stores the compiler can
        // wait for the prefetched loads alone (stores share the vector-memory
        // counter), instead of draining every store of the tile
#pragma unroll
        for (int grp = 0; grp < 8; ++grp) {
            v4f acc[4];
            mlp.layer1(f, acc);
            float fn[8];
            if (grp < 7) perceive_2d(pl, tapw, g, centre_of(grp + 1), cb, fn);
            const v4f u = mlp.layer2(acc);

            const int r = grp >> 1;                 // row slot within the wave
            const int ly = 4 * wave + r;
            const int y = y0 + ly, x = x0 + (grp & 1) * 16 + n;
            const uint64_t idx = (uint64_t)y * dw + x;
            const uint64_t row_b0 = ((uint64_t)y * dw + x0) >> 3;
            const uint32_t off = x < dw ? (uint32_t)ly * row_bytes + (uint32_t)x * kCellBytes : kOut;
            update_store<Mlp>(dst, wr, off, g, f, u, fire.bit(slot0 + r, idx, row_b0));
#pragma unroll
            for (int k = 0; k < 8; ++k) f[k] = fn[k];
            // keep the scheduler from interleaving whole groups (register pressure)
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        ld.commit(planes);   // the next tile (zeros when there is none)
    }
}

// ---------------------------------------------------------------------------
// 2D, row streaming: a block is one wave, and a work item is a 32-cell-wide
// strip of a run of rows.  The wave streams the strip's halo rows (34 cells)
// through a private ring of four LDS row slots, so no block barrier is
// needed (LDS accesses of one wave complete in order).  Each input row q is
// read once: its 3 taps along x feed three rolling perception sums per
// 16-cell group, for outputs q + 1 (the dy = -1 weights), q (dy = 0) and
// q - 1 (dy = +1).  After row q the sum of output q - 1 is complete and that
// row's MLP, fire gate and store run, with the cell's own state re-read from
// the ring.  An iteration takes two input rows; the loads of the next two are
// issued at its start and written to LDS at its end.
// ---------------------------------------------------------------------------
constexpr int k2RunRows = 128;      // output rows per work item
constexpr int k2WavesPerSimd = 2;   // 255 VGPRs with the split-bf16 MLP

// The row kernels' conv weights: tapw[t][q] = the tap-t weights of channels
// 4q..4q+3 and cb = the bias of the lane's channel quad, both times the MLP's
// perception scale (Sec. 3.1: one 3x3 filter and bias per channel).  Quads
// >= C / 4 (quad 3 of a C = 12 model) are zero; their indices are clamped and
// the values replaced, so every lane loads.
template <int C>
__device__ __forceinline__ void load_conv_2d(const float *__restrict__ conv_w,
                                             const float *__restrict__ conv_b, float ps,
                                             float4 (*tapw)[4], float cb[4]) {
    const int lane = threadIdx.x & 63;
    const int i = lane % (9 * 4);
    const int t = i / 4, q = i % 4;
    const bool q_ok = q < C / 4;
    const int qc = q_ok ? q : 0;
    const float4 tw = make_float4(ps * conv_w[(4 * qc + 0) * 9 + t], ps * conv_w[(4 * qc + 1) * 9 + t],
                                  ps * conv_w[(4 * qc + 2) * 9 + t], ps * conv_w[(4 * qc + 3) * 9 + t]);
    const int g = lane >> 4;
    const bool g_ok = g < C / 4;
    const int gc = g_ok ? g : 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) cb[k] = g_ok ? ps * conv_b[4 * gc + k] : 0.f;
    // lanes >= 36 write an entry again with the same value: no branch, so the
    // loads above are not sunk behind one and wait once together
    tapw[t][q] = q_ok ? tw : make_float4(0.f, 0.f, 0.f, 0.f);
}

// One halo row of a strip: kBody body loads (16 cells x 4 chunks in fp32,
// 32 cells x 2 chunks in fp16, lane i -> cell i % cells-per-load, chunk
// i / cells-per-load) and one side load whose first 2 NQ lanes take the left
// and right halo cells.  Cells outside the grid and rows outside [0, h) read
// as zero through an out-of-range offset or an empty descriptor.  A cell of C
// channels fills kChunks of the NQ chunks; the others (channel quad 3 when
// C = 12) read as zero the same way, so the ring holds the cell padded to 16
// channels with zeros.
template <typename T, int C = kC>
struct RowStream {
    using Ch = CellChunk<T, C>;
    static constexpr int NQ = Ch::N;
    static constexpr int kCellBytes = C * (int)sizeof(T);
    static constexpr int kChunks = Ch::kUsed;
    static constexpr int kCellsPerBody = 64 / NQ;
    static constexpr int kBody = kTileW / kCellsPerBody;
    static constexpr int kDummy = kHaloW;                 // never-read slot
    static constexpr int PS = plane_stride(kHaloW + 1);   // quad plane stride (16-byte words)
    static constexpr int kSlotWords = 4 * PS;             // one ring slot
    uint4 v[kBody + 1];

    __device__ __forceinline__ void issue(const T *__restrict__ src, int y, int dh, int dw, int x0) {
        const int lane = threadIdx.x & 63;
        const bool row_ok = y >= 0 && y < dh;
        const Rsrc r = make_rsrc(src + (int64_t)(row_ok ? y : 0) * dw * C,
                                 row_ok ? (uint32_t)dw * kCellBytes : 0u);
        const int cell = lane % kCellsPerBody, chunk = lane / kCellsPerBody;
#pragma unroll
        for (int k = 0; k < kBody; ++k) {
            const int cx = x0 + k * kCellsPerBody + cell;
            const uint32_t off = chunk < kChunks && cx >= 0 && cx < dw
                                     ? (uint32_t)cx * kCellBytes + (uint32_t)chunk * Ch::kBytes
                                     : kOut;
            v[k] = Ch::load(r, off);
        }
        const int cx = lane < NQ ? x0 - 1 : x0 + kTileW;
        const bool ok = lane < 2 * NQ && lane % NQ < kChunks && cx >= 0 && cx < dw;
        const uint32_t off = ok ? (uint32_t)cx * kCellBytes + (uint32_t)(lane % NQ) * Ch::kBytes : kOut;
        v[kBody] = Ch::load(r, off);
    }

    // LDS: four channel-quad planes of PS 16-byte words, fp32; slot 0 is the
    // left halo cell, 1..32 the strip, 33 the right halo cell.
    __device__ static __forceinline__ void put(float4 *planes, int q, int slot, const uint4 &c) {
        Ch::put(planes, PS, q, slot, c);
    }

    __device__ __forceinline__ void commit(float4 *planes) const {
        const int lane = threadIdx.x & 63;
        const int cell = lane % kCellsPerBody, chunk = lane / kCellsPerBody;
#pragma unroll
        for (int k = 0; k < kBody; ++k) put(planes, chunk, 1 + k * kCellsPerBody + cell, v[k]);
        const int slot = lane < NQ ? 0 : (lane < 2 * NQ ? kHaloW - 1 : kDummy);
        put(planes, lane % NQ, slot, v[kBody]);
    }

    // Upsample + inject fused into the load (Sec. 3.2; supplement S6): fine row
    // y comes from the coarse state's row y / fy, cell x from coarse cell x / fx,
    // and the NIN input channels from the fine image's row y (one image element
    // per lane, kImg loads).  commit_up writes the coarse cells like commit()
    // and then overwrites the input channels (all in channel quad 0) with the
    // image values, so the ring holds exactly the upsampled fine state.
    template <int NIN>
    struct Image {
        static constexpr int kElems = kHaloW * NIN;
        static constexpr int kImg = (kElems + 63) / 64;
        uint32_t e[kImg];
    };

    template <int NIN>
    __device__ __forceinline__ void issue_up(const T *__restrict__ coarse, int cdw, int fy,
                                             int fx, const T *__restrict__ img, Image<NIN> &im,
                                             int y, int dh, int dw, int x0) {
        const int lane = threadIdx.x & 63;
        const bool row_ok = y >= 0 && y < dh;
        const Rsrc r = make_rsrc(coarse + (int64_t)(row_ok ? y / fy : 0) * cdw * C,
                                 row_ok ? (uint32_t)cdw * kCellBytes : 0u);
        const int cell = lane % kCellsPerBody, chunk = lane / kCellsPerBody;
#pragma unroll
        for (int k = 0; k < kBody; ++k) {
            const int cx = x0 + k * kCellsPerBody + cell;
            const uint32_t off = chunk < kChunks && cx >= 0 && cx < dw
                                     ? (uint32_t)(cx / fx) * kCellBytes + (uint32_t)chunk * Ch::kBytes
                                     : kOut;
            v[k] = Ch::load(r, off);
        }
        {
            const int cx = lane < NQ ? x0 - 1 : x0 + kTileW;
            const bool ok = lane < 2 * NQ && lane % NQ < kChunks && cx >= 0 && cx < dw;
            const uint32_t off =
                ok ? (uint32_t)(cx / fx) * kCellBytes + (uint32_t)(lane % NQ) * Ch::kBytes : kOut;
            v[kBody] = Ch::load(r, off);
        }
        const Rsrc ri = make_rsrc(img + (int64_t)(row_ok ? y : 0) * dw * NIN,
                                  row_ok ? (uint32_t)dw * NIN * (uint32_t)sizeof(T) : 0u);
#pragma unroll
        for (int j = 0; j < Image<NIN>::kImg; ++j) {
            const int e = lane + 64 * j;
            const int fc = x0 - 1 + e / NIN;
            const bool ok = e < Image<NIN>::kElems && fc >= 0 && fc < dw;
            const uint32_t off = ok ? (uint32_t)(fc * NIN + e % NIN) * (uint32_t)sizeof(T) : kOut;
            if constexpr (sizeof(T) == 4)
                im.e[j] = __builtin_amdgcn_raw_buffer_load_b32(ri, off, 0, 0);
            else
                im.e[j] = __builtin_amdgcn_raw_buffer_load_b16(ri, off, 0, 0);
        }
    }

    template <int NIN>
    __device__ __forceinline__ void commit_up(float4 *planes, const Image<NIN> &im) const {
        commit(planes);
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int j = 0; j < Image<NIN>::kImg; ++j) {
            const int e = lane + 64 * j;
            const int slot = e < Image<NIN>::kElems ? e / NIN : kDummy;
            float val;
            if constexpr (sizeof(T) == 4)
                val = __uint_as_float(im.e[j]);
            else
                val = __half2float(__ushort_as_half((unsigned short)im.e[j]));
            reinterpret_cast<float *>(planes + slot)[e % NIN] = val;   // quad plane 0
        }
    }
};

// UP: the step's input is not a state of this level but the next coarser
// level's state (src, width up_cdw) upsampled by (up_fy, up_fx) with the input
// channels taken from up_img (the first step of a level, fused with the
// upsample + inject).
template <typename T, int NIN, class Mlp, bool ALIGNED, bool UP>
__global__ __launch_bounds__(64, k2WavesPerSimd) void nca_step_mfma_2d_rows(
    const T *__restrict__ src, T *__restrict__ dst, int dh, int dw, int strips, int runs,
    int run_rows, int items, const float *__restrict__ conv_w,
    const float *__restrict__ conv_b, const float *__restrict__ w1, const float *__restrict__ b1,
    const float *__restrict__ w2, uint32_t level, uint32_t step, uint32_t batch, uint64_t seed,
    uint64_t threshold, const T *__restrict__ up_img, int up_cdw, int up_fy, int up_fx) {
    constexpr int C = Mlp::kChannels;
    using RS = RowStream<T, C>;
    __shared__ float4 ring[4][RS::kSlotWords];   // row y in slot y & 3
    __shared__ float4 tapw[9][4];                // [tap][quad] conv weights of channels 4q..4q+3

    const int lane = threadIdx.x & 63;
    const int n = lane & 15;
    const int g = lane >> 4;

    Mlp mlp;
    mlp.load(w1, b1, w2, n, g, NIN);
    float cb[4];
    load_conv_2d<C>(conv_w, conv_b, Mlp::kPerceptionScale, tapw, cb);
    mlp.pin_all();
#pragma unroll
    for (int k = 0; k < 4; ++k) pin(cb[k]);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    // Fire evaluations: a row takes opr lanes, so one evaluation serves
    // 64 / opr consecutive output rows (16 when rows are 8-aligned, else 8).
    // ALIGNED (w % 8 == 0): a lane's cells always take ballot n % 8 at bit
    // offset 2 grp + n / 8 within their row's slot.
    FireBits fire;
    fire.aligned = ALIGNED;
    fire.opr = ALIGNED ? 4 : 8;
    constexpr int lg_opr = ALIGNED ? 2 : 3;
    constexpr int rows_per_eval = ALIGNED ? 16 : 8;
    constexpr int kCellBytes = RS::kCellBytes;
    const uint32_t row_bytes = (uint32_t)dw * kCellBytes;
    int gq = g;
    RS ra, rb;
    typename RS::template Image<NIN> ia, ib;   // used by UP only
    // Rows at or beyond y_lim (the run's last input row + 1, or the grid's
    // height) read as zero through an empty descriptor, without a memory access.
    int y_lim = dh;
    auto issue = [&](RS &rs, typename RS::template Image<NIN> &im, int y, int x0) {
        if constexpr (UP)
            rs.template issue_up<NIN>(src, up_cdw, up_fy, up_fx, up_img, im, y, y_lim, dw, x0);
        else
            rs.issue(src, y, y_lim, dw, x0);
    };
    auto commit = [&](const RS &rs, const typename RS::template Image<NIN> &im, float4 *slot) {
        if constexpr (UP)
            rs.template commit_up<NIN>(slot, im);
        else
            rs.commit(slot);
    };

    for (int item = blockIdx.x; item < items; item += gridDim.x) {
        const int sx = item % strips;
        const int ry = item / strips;
        const int x0 = sx * kTileW;
        const int y_begin = ry * run_rows;
        const int y_end = min(dh, y_begin + run_rows);
        y_lim = min(dh, y_end + 1);   // input rows y_begin - 1 .. y_end feed the run

        // rolling perception sums (bias included) of outputs q - 1, q, q + 1
        float acc_p[2][4], acc_c[2][4], acc_n[2][4];
#pragma unroll
        for (int grp = 0; grp < 2; ++grp)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                acc_p[grp][k] = cb[k];
                acc_c[grp][k] = cb[k];
                acc_n[grp][k] = cb[k];
            }

        // Input row q with its x taps: output q + 1 takes the dy = -1 weights,
        // q the dy = 0 ones and q - 1 the dy = +1 ones.
        auto fold_row = [&](int q) {
            const float4 *pl = ring[q & 3] + g * RS::PS;
            pin(gq);   // re-read the tap weights every row instead of keeping 36 registers
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) {
                const float4 wm = tapw[dx][gq];
                const float4 w0 = tapw[3 + dx][gq];
                const float4 wp = tapw[6 + dx][gq];
                const float a_m[4] = {wm.x, wm.y, wm.z, wm.w};
                const float a_0[4] = {w0.x, w0.y, w0.z, w0.w};
                const float a_p[4] = {wp.x, wp.y, wp.z, wp.w};
#pragma unroll
                for (int grp = 0; grp < 2; ++grp) {
                    const float4 v = pl[grp * 16 + n + dx];
                    const float vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        acc_n[grp][k] = fmaf(a_m[k], vv[k], acc_n[grp][k]);
                        acc_c[grp][k] = fmaf(a_0[k], vv[k], acc_c[grp][k]);
                        acc_p[grp][k] = fmaf(a_p[k], vv[k], acc_p[grp][k]);
                    }
                }
            }
        };

        // Fire bits of output rows yo .. yo + rows_per_eval - 1.
        auto evaluate_fire = [&](int yo) {
            const int yy = min(yo + (lane >> lg_opr), dh - 1);
            const uint64_t b0 = ((uint64_t)yy * dw + x0) >> 3;
            fire.f = fire_ballots(b0 + (lane & (fire.opr - 1)), step, level, batch, seed, threshold);
            fire.mine = select_ballot(fire.f, (uint32_t)n & 7u);
        };

        // The sums shift by one row: output q + 1 becomes the next to finish.
        auto shift = [&]() {
#pragma unroll
            for (int grp = 0; grp < 2; ++grp)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    acc_p[grp][k] = acc_c[grp][k];
                    acc_c[grp][k] = acc_n[grp][k];
                    acc_n[grp][k] = cb[k];
                }
        };

        // Output row yo (complete in acc_p): MLP, fire gate and store of its
        // two groups; stores of rows outside [y_begin, y_end) are dropped by an
        // empty descriptor.  Then the sums shift by one row.
        auto finish_row = [&](int yo) {
            const bool out_ok = yo >= y_begin && yo < y_end;
            const int phase = (yo - y_begin) & (rows_per_eval - 1);
            if (out_ok && phase == 0 && yo != y_begin) evaluate_fire(yo);
            const int yc = max(yo, 0);
            const Rsrc wr = make_rsrc(dst + (int64_t)yc * dw * C, out_ok ? row_bytes : 0u);
            const float4 *own = ring[yo & 3] + g * RS::PS;
            const uint64_t row_b0 = ((uint64_t)yc * dw + x0) >> 3;
            v4f acc[2][4];
            float f[2][8];
#pragma unroll
            for (int grp = 0; grp < 2; ++grp) {
                const float4 sp = own[1 + grp * 16 + n];
                f[grp][0] = sp.x; f[grp][1] = sp.y; f[grp][2] = sp.z; f[grp][3] = sp.w;
#pragma unroll
                for (int k = 0; k < 4; ++k) f[grp][4 + k] = acc_p[grp][k];
                mlp.layer1(f[grp], acc[grp]);
            }
#pragma unroll
            for (int grp = 0; grp < 2; ++grp) {
                const v4f u = mlp.layer2(acc[grp]);
                const int x = x0 + grp * 16 + n;
                const uint32_t off = x < dw && g < C / 4 ? (uint32_t)x * kCellBytes : kOut;
                bool fires;
                if constexpr (ALIGNED) {
                    fires = (fire.mine >> (phase * 4 + 2 * grp + (n >> 3))) & 1;
                } else {
                    const uint64_t idx = (uint64_t)yc * dw + x;
                    fires = fire.bit(phase, idx, row_b0);
                }
                update_store<Mlp>(dst, wr, off, g, f[grp], u, fires);
            }
            shift();
        };

        // Rows y_begin - 1 and y_begin into the ring, y_begin + 1 and
        // y_begin + 2 in flight while they are folded; outputs y_begin - 2 and
        // y_begin - 1, which they complete, are outside the run (not computed).
        // The run's first fire evaluation runs while the first rows load.
        issue(ra, ia, y_begin - 1, x0);
        issue(rb, ib, y_begin, x0);
        evaluate_fire(y_begin);
        commit(ra, ia, ring[(y_begin - 1) & 3]);
        commit(rb, ib, ring[y_begin & 3]);
        issue(ra, ia, y_begin + 1, x0);
        issue(rb, ib, y_begin + 2, x0);
        fold_row(y_begin - 1);
        shift();
        fold_row(y_begin);
        shift();
        commit(ra, ia, ring[(y_begin + 1) & 3]);
        commit(rb, ib, ring[(y_begin + 2) & 3]);

        // input rows q, q + 1 per iteration, from y_begin + 1 through y_end
        // (plus one padding row when the count is odd)
        for (int q = y_begin + 1; q <= y_end; q += 2) {
            issue(ra, ia, q + 2, x0);
            issue(rb, ib, q + 3, x0);
            fold_row(q);
            finish_row(q - 1);
            __builtin_amdgcn_sched_barrier(0);
            fold_row(q + 1);
            finish_row(q);
            __builtin_amdgcn_sched_barrier(0);
            commit(ra, ia, ring[(q + 2) & 3]);
            commit(rb, ib, ring[(q + 3) & 3]);
        }
    }
}

// ---------------------------------------------------------------------------
// 2D, two steps per launch (temporal fusion).  The fire mask is a function of
// (seed, level, step, cell) alone, so a wave can run step t + 1 on its own
// copy of step t's result.  Same row streaming as nca_step_mfma_2d_rows, with
// the strip narrowed to 30 output cells: the wave loads 34-cell halo rows
// (cells x0 - 2 .. x0 + 31), runs step t on the 32 cells x0 - 1 .. x0 + 30 and
// writes each finished row into a second LDS ring of two slots (cells and
// rows outside the grid as 0: the zero padding of step t + 1's perception).
// Step t + 1 folds those rows into its own rolling sums and finishes cells
// x0 .. x0 + 31, of which x0 .. x0 + 29 are stored (the last two lack their
// right neighbours).  Per input row q: step t folds q and finishes q - 1, then
// step t + 1 folds q - 1; its row q - 2, complete then, is finished in the
// next row's body, next to step t's fold.  The state between the two steps
// never reaches HBM, so HBM sees one read and one write of the state per two
// steps, for 32/30 of the MLP work and 2 halo rows of step t per run; the
// results equal two single-step launches bit for bit (the same operations in
// the same order).
// ---------------------------------------------------------------------------
constexpr int k2PairW = kTileW - 2;   // output cells per strip

// UP: step t is a level's first step, fused with the upsample + inject as in
// nca_step_mfma_2d_rows (src is the next coarser state, width up_cdw, factors
// up_fy, up_fx; the input channels come from up_img).  SEG: the launch also
// writes the two-class readout of its result (Sec. 3.2) to seg: the lanes of
// channel quad 3 hold channels 12..15 of their cell, and its byte is 1 iff
// channel C - 1 > channel C - 2 (ties and NaNs give 0), the readout kernel's
// rule; the finest level's last launch uses it.
template <typename T, int NIN, class Mlp, bool UP, bool SEG>
__global__ __launch_bounds__(64, k2WavesPerSimd) void nca_step2_mfma_2d_rows(
    const T *__restrict__ src, T *__restrict__ dst, int dh, int dw, int strips, int run_rows,
    int items, const float *__restrict__ conv_w, const float *__restrict__ conv_b,
    const float *__restrict__ w1, const float *__restrict__ b1, const float *__restrict__ w2,
    uint32_t level, uint32_t step, uint32_t batch, uint64_t seed, uint64_t threshold,
    const T *__restrict__ up_img, int up_cdw, int up_fy, int up_fx, uint8_t *__restrict__ seg) {
    static_assert(std::is_same_v<T, float>, "the intermediate ring holds fp32 states");
    constexpr int C = Mlp::kChannels;
    using RS = RowStream<T, C>;
    // Row r of a work item (first input row `base`) lives in slot
    // (r - base) % 3 of the input ring and (r - base) % 2 of the ring of step
    // t's output rows.
    __shared__ float4 ring[3][RS::kSlotWords];
    __shared__ float4 mid[2][RS::kSlotWords];
    __shared__ float4 tapw[9][4];                // [tap][quad] conv weights of channels 4q..4q+3
    // Fire bits of the work item, [step t / t + 1][row]: byte o of a row's
    // word holds the 8 draws of the o-th block of 8 cells from the block that
    // contains the row's first strip cell.
    constexpr int kOpr = 5, kEvalRows = 12;
    constexpr int kEvalBlocks = (k2RunRows + 2 + kEvalRows - 1) / kEvalRows;
    constexpr int kMaskRows = kEvalBlocks * kEvalRows;
    __shared__ uint64_t fire_rows[2][kMaskRows];
    // The same words shifted once per work item so that bit c is the draw of
    // strip cell c (x0 - 1 + c for step t, x0 + c for step t + 1): a lane's
    // bit is then one bit-field extract.
    __shared__ uint32_t fire_bits[2][kMaskRows];

    const int lane = threadIdx.x & 63;
    const int n = lane & 15;
    const int g = lane >> 4;

    // Slots 32 and 33 of the step-t ring are never written: the two cells
    // per quad that step t + 1 computes but does not store read them.
    if (lane < 16) mid[lane >> 3][((lane >> 1) & 3) * RS::PS + 32 + (lane & 1)] = make_float4(0.f, 0.f, 0.f, 0.f);
    Mlp mlp;
    mlp.load(w1, b1, w2, n, g, NIN);
    float cb[4];
    load_conv_2d<C>(conv_w, conv_b, Mlp::kPerceptionScale, tapw, cb);
    mlp.pin_all();
#pragma unroll
    for (int k = 0; k < 4; ++k) pin(cb[k]);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    // Fire evaluations: a strip row spans at most 5 blocks of 8 cells (it may
    // start anywhere within a block), so an evaluation gives 5 lanes to each of
    // 12 rows of one step (lanes 60..63 repeat row 11).  All evaluations of a
    // work item run at its start, where few registers are live; each lane
    // writes the 8 fire bits of its block as one byte of its row's word.
    const int ev_row = min(lane / kOpr, kEvalRows - 1), ev_blk = lane % kOpr;
    auto evaluate = [&](int s, int blk, uint32_t st, int y_first, uint32_t xs) {
        const int yy = min(max(y_first + ev_row, 0), dh - 1);
        const uint64_t b0 = (((uint64_t)yy * dw + xs) >> 3) + ev_blk;
        const Philox4x64Out r = philox4x64_10(b0, st, level, batch, seed, 0);
        uint32_t bits = 0;
#pragma unroll
        for (int c = 0; c < 8; ++c) bits |= ((uint64_t)draw_of(r, (uint32_t)c) < threshold ? 1u : 0u) << c;
        reinterpret_cast<uint8_t *>(&fire_rows[s][blk * kEvalRows + ev_row])[ev_blk] = (uint8_t)bits;
    };
    // Fire bit of strip cell c (c = x - xs >= 0) in row `rel` (rows from the
    // step's first row) of step s, whose row starts at canonical index rowc:
    // bit c + ((rowc + xs) & 7) of the row's word in fire_rows, bit c of its
    // word in fire_bits.  2D cell indices fit 32 bits (two fp32 states of
    // 2^32 cells would need 512 GB).  Rows outside the step's range read some
    // in-range word.
    auto row_bits = [&](int s, int rel) {
        return fire_bits[s][min(max(rel, 0), kMaskRows - 1)];
    };
    constexpr int kCellBytes = RS::kCellBytes;
    const uint32_t row_bytes = (uint32_t)dw * kCellBytes;
    int gq = g;
    RS ra, rb;
    using Img = typename RS::template Image<NIN>;
    Img ia, ib;   // used by UP only
    // UP: the lane's byte offsets within a coarse row and an image row, the
    // same for every row of a work item (computed once per item).
    struct UpCols {
        uint32_t body[RS::kBody], side, img[Img::kImg];
    } uc;
    auto up_cols = [&](int x) {
        const int lane = threadIdx.x & 63;
        const int cell = lane % RS::kCellsPerBody, chunk = lane / RS::kCellsPerBody;
#pragma unroll
        for (int kk = 0; kk < RS::kBody; ++kk) {
            const int cx = x + kk * RS::kCellsPerBody + cell;
            uc.body[kk] = chunk < RS::kChunks && cx >= 0 && cx < dw
                              ? (uint32_t)(cx / up_fx) * kCellBytes + (uint32_t)chunk * RS::Ch::kBytes : kOut;
        }
        const int cx = lane < RS::NQ ? x - 1 : x + kTileW;
        uc.side = lane < 2 * RS::NQ && lane % RS::NQ < RS::kChunks && cx >= 0 && cx < dw
                      ? (uint32_t)(cx / up_fx) * kCellBytes + (uint32_t)(lane % RS::NQ) * RS::Ch::kBytes : kOut;
#pragma unroll
        for (int j = 0; j < Img::kImg; ++j) {
            const int e = lane + 64 * j;
            const int fc = x - 1 + e / NIN;
            uc.img[j] = e < Img::kElems && fc >= 0 && fc < dw
                            ? (uint32_t)(fc * NIN + e % NIN) * (uint32_t)sizeof(T) : kOut;
        }
    };
    // Fine row y of the upsampled state: coarse row cy = y / fy, image row y.
    // The loop passes cy kept by counting (a division per row in the unrolled
    // loop made the compiler spill).
    auto issue = [&](RS &rs, Img &im, int y, int cy, int x) {
        if constexpr (UP) {
            const bool row_ok = y >= 0 && y < dh;
            const Rsrc r = make_rsrc(src + (int64_t)(row_ok ? cy : 0) * up_cdw * C,
                                     row_ok ? (uint32_t)up_cdw * kCellBytes : 0u);
#pragma unroll
            for (int kk = 0; kk < RS::kBody; ++kk) {
                const v4u v = __builtin_amdgcn_raw_buffer_load_b128(r, uc.body[kk], 0, 0);
                rs.v[kk] = make_uint4(v[0], v[1], v[2], v[3]);
            }
            const v4u v = __builtin_amdgcn_raw_buffer_load_b128(r, uc.side, 0, 0);
            rs.v[RS::kBody] = make_uint4(v[0], v[1], v[2], v[3]);
            const Rsrc ri = make_rsrc(up_img + (int64_t)(row_ok ? y : 0) * dw * NIN,
                                      row_ok ? (uint32_t)dw * NIN * (uint32_t)sizeof(T) : 0u);
#pragma unroll
            for (int j = 0; j < Img::kImg; ++j)
                im.e[j] = __builtin_amdgcn_raw_buffer_load_b32(ri, uc.img[j], 0, 0);
        } else {
            rs.issue(src, y, dh, dw, x);
        }
    };
    auto commit = [&](const RS &rs, const Img &im, float4 *slot) {
        if constexpr (UP)
            rs.template commit_up<NIN>(slot, im);
        else
            rs.commit(slot);
    };

    for (int item = blockIdx.x; item < items; item += gridDim.x) {
        const int sx = item % strips;
        const int ry = item / strips;
        const int x0 = sx * k2PairW;
        const int x1 = x0 - 1;             // first cell of step t's strip
        const uint32_t xs1 = (uint32_t)max(x1, 0);
        const int y_begin = ry * run_rows;
        const int y_end = min(dh, y_begin + run_rows);
        const int x_stop = min(dw, x0 + k2PairW);
        const int base = y_begin - 2;      // first input row

        // Rolling perception sums (bias included): A[(r - base) % 3] holds
        // step t's sum of output row r, B[(r - base) % 3] step t + 1's.  The
        // loop body is unrolled three times, so the three sums of a step
        // rotate roles without register moves.
        float A[3][2][4], B[3][2][4];

        if constexpr (UP) up_cols(x1);
        issue(ra, ia, base, base >= 0 ? base / up_fy : 0, x1);
        issue(rb, ib, base + 1, base + 1 >= 0 ? (base + 1) / up_fy : 0, x1);
        // coarse row and remainder of the next row the loop loads (y_begin >= 0)
        int up_cy = y_begin / up_fy, up_ry = y_begin - up_cy * up_fy;
        // step t's rows y_begin - 1 .. y_end, step t + 1's y_begin .. y_end - 1
        for (int e = 0; e < 2 * kEvalBlocks; ++e) {
            const int st = e >= kEvalBlocks ? 1 : 0;
            const int blk = e - st * kEvalBlocks;
            const int y_first = y_begin - 1 + st + blk * kEvalRows;
            if (y_first <= y_end - st)
                evaluate(st, blk, step + st, y_first, st ? (uint32_t)x0 : xs1);
        }
        // Align each row's word to the strip: step t's strip starts at x1
        // (x1 = -1 on the first strip, whose cell 0 is outside the grid and
        // gets bit 0, unused), step t + 1's at x0.  A word spans the 5 blocks
        // of 8 cells that hold cells xs .. xs + 31, so bits sh .. sh + 31 with
        // sh <= 7 are inside it.
        for (int i = lane; i < 2 * kMaskRows; i += 64) {
            const int s = i >= kMaskRows ? 1 : 0;
            const int rel = i - s * kMaskRows;
            const int yo = y_begin - 1 + s + rel;
            const uint32_t rowc = (uint32_t)min(max(yo, 0), dh - 1) * (uint32_t)dw;
            const int sh = s ? (int)((rowc + (uint32_t)x0) & 7u)
                             : (int)((rowc + xs1) & 7u) + (x1 - (int)xs1);
            fire_bits[s][rel] = (uint32_t)((fire_rows[s][rel] << 1) >> (sh + 1));
        }
        commit(ra, ia, ring[0]);
        commit(rb, ib, ring[1]);

        // Row r of a plane set with its x taps: output r + 1 takes the dy = -1
        // weights (its first contribution, started from the bias), r the
        // dy = 0 ones and r - 1 the dy = +1 ones (its last).
        auto fold = [&](const float4 *pl, float (&first)[2][4], float (&second)[2][4],
                        float (&last)[2][4]) {
            pin(gq);   // re-read the tap weights every row instead of keeping 36 registers
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) {
                const float4 wm = tapw[dx][gq];
                const float4 w0 = tapw[3 + dx][gq];
                const float4 wp = tapw[6 + dx][gq];
                const float a_m[4] = {wm.x, wm.y, wm.z, wm.w};
                const float a_0[4] = {w0.x, w0.y, w0.z, w0.w};
                const float a_p[4] = {wp.x, wp.y, wp.z, wp.w};
#pragma unroll
                for (int grp = 0; grp < 2; ++grp) {
                    const float4 v = pl[grp * 16 + n + dx];
                    const float vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        first[grp][k] = fmaf(a_m[k], vv[k], dx == 0 ? cb[k] : first[grp][k]);
                        second[grp][k] = fmaf(a_0[k], vv[k], second[grp][k]);
                        last[grp][k] = fmaf(a_p[k], vv[k], last[grp][k]);
                    }
                }
            }
        };

        // Step t, row yo (complete in p) -> mid ring.  Rows y_begin - 1 ..
        // y_end are the ones step t + 1 reads; earlier rows are pipeline
        // start-up whose values are never used.
        auto finish_a = [&](int yo, int slot, const float (&p)[2][4]) {
            const bool row_in = yo >= 0 && yo < dh;
            const uint32_t fl = row_bits(0, yo - (y_begin - 1)) >> n;   // bits 0, 16: cells n, 16 + n
            const float4 *own = ring[slot] + g * RS::PS;
            float4 *out = mid[(yo - base) & 1] + g * RS::PS;
            v4f acc[2][4];
            float f[2][8];
#pragma unroll
            for (int grp = 0; grp < 2; ++grp) {
                const float4 sv = own[1 + grp * 16 + n];
                f[grp][0] = sv.x; f[grp][1] = sv.y; f[grp][2] = sv.z; f[grp][3] = sv.w;
#pragma unroll
                for (int k = 0; k < 4; ++k) f[grp][4 + k] = p[grp][k];
                mlp.layer1(f[grp], acc[grp]);
            }
#pragma unroll
            for (int grp = 0; grp < 2; ++grp) {
                const v4f u = mlp.layer2(acc[grp]);
                const int x = x1 + grp * 16 + n;
                const bool in = row_in && x >= 0 && x < dw;
                const float m = (float)__builtin_amdgcn_ubfe(fl, grp * 16u, 1u);
                float v[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) v[k] = in ? fmaf(m, u[k], f[grp][k]) : 0.f;
                out[grp * 16 + n] = make_float4(v[0], v[1], v[2], v[3]);
            }
        };

        // Step t + 1, row yo (complete in p): MLP, fire gate and store; rows
        // outside [y_begin, y_end) are dropped by an empty descriptor.
        auto finish_b = [&](int yo, const float (&p)[2][4]) {
            const bool out_ok = yo >= y_begin && yo < y_end;
            const int yc = min(max(yo, 0), dh - 1);
            const uint32_t fl = row_bits(1, yo - y_begin) >> n;   // bits 0, 16: cells n, 16 + n
            const Rsrc wr = make_rsrc(dst + (int64_t)yc * dw * C, out_ok ? row_bytes : 0u);
            const float4 *own = mid[(yo - base) & 1] + g * RS::PS;
            v4f acc[2][4];
            float f[2][8];
#pragma unroll
            for (int grp = 0; grp < 2; ++grp) {
                const float4 sv = own[1 + grp * 16 + n];
                f[grp][0] = sv.x; f[grp][1] = sv.y; f[grp][2] = sv.z; f[grp][3] = sv.w;
#pragma unroll
                for (int k = 0; k < 4; ++k) f[grp][4 + k] = p[grp][k];
                mlp.layer1(f[grp], acc[grp]);
            }
#pragma unroll
            for (int grp = 0; grp < 2; ++grp) {
                const v4f u = mlp.layer2(acc[grp]);
                const int x = x0 + grp * 16 + n;
                const uint32_t off = x < x_stop && g < C / 4 ? (uint32_t)x * kCellBytes : kOut;
                const float m = (float)__builtin_amdgcn_ubfe(fl, grp * 16u, 1u);
                if constexpr (SEG) {
                    v4f o;
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) o[kk] = fmaf(m, u[kk], f[grp][kk]);
                    store_quad(dst, wr, off, g, o);
                    const Rsrc sr = make_rsrc(seg + (int64_t)yc * dw, out_ok ? (uint32_t)dw : 0u);
                    const uint32_t so = g == C / 4 - 1 && x < x_stop ? (uint32_t)x : kOut;
                    __builtin_amdgcn_raw_buffer_store_b8((unsigned char)(o[3] > o[2] ? 1 : 0), sr,
                                                         so, 0, 0);
                } else {
                    update_store<Mlp>(dst, wr, off, g, f[grp], u, m);
                }
            }
        };

        // One input row q per body, from base through y_end + 1 (rounded up
        // to whole groups of three): step t finishes row q - 1, step t + 1 row
        // q - 2.  Row q + 2 is loaded during the body and written to the slot
        // of row q - 1 at its end.
        auto body = [&](int q, auto jc) {
            constexpr int j = decltype(jc)::value;   // (q - base) % 3
            constexpr int jm = (j + 2) % 3, jp = (j + 1) % 3;   // rows q - 1, q + 1 (= q - 2)
            issue(ra, ia, q + 2, up_cy, x1);
            if constexpr (UP) {
                up_cy += ++up_ry == up_fy ? 1 : 0;
                up_ry = up_ry == up_fy ? 0 : up_ry;
            }
            // input row q: outputs q + 1, q, q - 1 of step t; next to it
            // (independent, so the matrix cores overlap the fold's FMAs) step
            // t + 1's row q - 3, whose sum the previous body completed (B[j]
            // is restarted by this body's second fold)
            fold(ring[j] + g * RS::PS, A[jp], A[j], A[jm]);
            finish_b(q - 3, B[j]);
            finish_a(q - 1, jm, A[jm]);
            __builtin_amdgcn_sched_barrier(0);
            // step t's row q - 1: outputs q, q - 1, q - 2 of step t + 1
            fold(mid[(q - 1 - base) & 1] + g * RS::PS, B[j], B[jm], B[jp]);
            __builtin_amdgcn_sched_barrier(0);
            commit(ra, ia, ring[jm]);
        };
        // The first bodies see sums that were never started (rows before
        // base); they only feed rows that are not used.
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int grp = 0; grp < 2; ++grp)
#pragma unroll
                for (int k = 0; k < 4; ++k) A[i][grp][k] = B[i][grp][k] = cb[k];
        int q0 = base;
        for (; q0 <= y_end + 1; q0 += 3) {
            body(q0, std::integral_constant<int, 0>{});
            body(q0 + 1, std::integral_constant<int, 1>{});
            body(q0 + 2, std::integral_constant<int, 2>{});
        }
        finish_b(q0 - 3, B[0]);   // the last body's deferred row
    }
}

// ---------------------------------------------------------------------------
// 3D: a work item is an 8 x 32 (y, x) column and a run of `zrun` output
// planes (up to k3ZRun; the launch picks it with a load model).  Input planes
// stream through a ring of three LDS plane slots
// (planes p - 1 and p are in use while p + 1 is written).  Each input plane p
// is read once: its 9 in-plane taps feed three rolling perception sums, for
// outputs p + 1 (the dz = -1 weights), p (dz = 0) and p - 1 (dz = +1).  After
// plane p the sum of output p - 1 is complete and that plane's MLP, fire gate
// and store run, with the cell's own state re-read from the ring.  Wave w
// owns rows 2w, 2w+1 (4 groups of 16 cells); the conv weights of a tap are
// read once per wave and applied to all 4 groups.
// ---------------------------------------------------------------------------
constexpr int k3TY = 8;
// Longest run of output planes per work item.  A run re-reads two halo planes,
// so long runs on deep levels stream less; its fire words (one evaluation per
// 4 or 8 planes) take k3ZRun / 4 x 64 B of LDS per wave.  128 keeps 2 blocks
// per CU (78 KB each).
constexpr int k3ZRun = 128;
// Work item i of a 3D step is tile (tx, ty) of z run zr, with
// i = (zr * tiles_y + ty) * tiles_x + tx.

// ALIGNED: rows start on an 8-cell boundary (w % 8 == 0), which makes the
// ballot and the bit offset of a lane's cells lane constants.
template <typename T, int NIN, class Mlp, bool ALIGNED>
__global__ __launch_bounds__(kThreads, 2) void nca_step_mfma_3d(
    const T *__restrict__ src, T *__restrict__ dst, int dd, int dh, int dw, int tiles_x,
    int tiles_y, int items, int zrun, const float *__restrict__ conv_w,
    const float *__restrict__ conv_b,
    const float *__restrict__ w1, const float *__restrict__ b1, const float *__restrict__ w2,
    uint32_t level, uint32_t step, uint32_t batch, uint64_t seed, uint64_t threshold) {
    // C = 16 (H = 64) or the ablation's C = 12 (H = 48): channel quad 3 idle
    constexpr int C = Mlp::kChannels;
    using Loader = RowLoader<T, k3TY + 2, C>;
    __shared__ float4 ring[3][4 * Loader::PS];
    __shared__ float4 tapw[27][4];      // [tap][quad] conv weights of channels 4q..4q+3
    // [wave][evaluation of the work item][b]: ballot b (k3ZRun / 4 evaluations
    // at most: one per 4 or 8 planes)
    __shared__ uint64_t fire_words[4][k3ZRun / 4][8];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15;
    const int g = lane >> 4;

    {
        const int i = min((int)threadIdx.x, 27 * 4 - 1);
        const int t = i / 4, q = i % 4;
        const int qc = q < C / 4 ? q : 0;   // quads >= C / 4: zero weights
        constexpr float ps = Mlp::kPerceptionScale;
        const float4 tw = make_float4(ps * conv_w[(4 * qc + 0) * 27 + t], ps * conv_w[(4 * qc + 1) * 27 + t],
                                      ps * conv_w[(4 * qc + 2) * 27 + t], ps * conv_w[(4 * qc + 3) * 27 + t]);
        if (threadIdx.x < 27 * 4) tapw[t][q] = q < C / 4 ? tw : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    Mlp mlp;
    mlp.load(w1, b1, w2, n, g, NIN);
    float cb[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        cb[k] = g < C / 4 ? Mlp::kPerceptionScale * conv_b[4 * (g < C / 4 ? g : 0) + k] : 0.f;
    mlp.pin_all();
#pragma unroll
    for (int k = 0; k < 4; ++k) pin(cb[k]);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    // Fire evaluations: a plane's 2 rows per wave take 2 * opr lanes, so one
    // evaluation serves 64 / (2 opr) consecutive output planes (8 when rows
    // are 8-aligned, else 4).  The 8 ballots go to a per-wave LDS array and a
    // cell reads the one it needs by address: selecting among them by a
    // per-lane value in registers makes the compiler build a private
    // (scratch) array, whose loads would be waited for with the stores.
    constexpr int opr = ALIGNED ? 4 : 8;
    constexpr int lg_opr = ALIGNED ? 2 : 3;
    constexpr int planes_per_eval = 64 / (2 * opr);
    constexpr int kCellBytes = Loader::kCellBytes;
    const uint32_t row_bytes = (uint32_t)dw * kCellBytes;
    Loader ld;
    // LDS word of group grp's cell (row 2 wave + grp / 2, column 16 (grp % 2) + n)
    // in the quad plane of this lane, relative to a plane slot.
    int centre[4];
#pragma unroll
    for (int grp = 0; grp < 4; ++grp)
        centre[grp] = g * Loader::PS + (2 * wave + (grp >> 1) + 1) * kHaloW + (grp & 1) * 16 + n + 1;

    const int64_t span = ((int64_t)items + gridDim.x - 1) / gridDim.x * gridDim.x;
    for (int64_t u = blockIdx.x; u < span; u += gridDim.x) {
        const int64_t it = xcd_item(u, (int)gridDim.x);
        if (it >= items) continue;                       // uniform over the block
        const int tiles = tiles_x * tiles_y;
        const int zr = (int)it / tiles;
        const int rest = (int)it - zr * tiles;
        const int tx = rest % tiles_x;
        const int ty = rest / tiles_x;
        const int y0 = ty * k3TY, x0 = tx * kTileW;
        const int z_begin = zr * zrun;
        const int z_end = min(dd, z_begin + zrun);
        // store offsets of the lane's 4 cells within an output plane's tile rows
        uint32_t offs[4];
#pragma unroll
        for (int grp = 0; grp < 4; ++grp) {
            const int x = x0 + (grp & 1) * 16 + n;
            offs[grp] = x < dw && g < C / 4
                            ? (uint32_t)(2 * wave + (grp >> 1)) * row_bytes + (uint32_t)x * kCellBytes
                            : kOut;
        }

        // Rolling perception sums (bias included): A[(r - z_begin + 1) % 3]
        // holds the sum of output plane r.  The plane loop is unrolled three
        // times, so the sums rotate roles instead of being moved; a run is
        // padded to whole groups of three planes (padding planes load and
        // store nothing).
        float A[3][4][4];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int grp = 0; grp < 4; ++grp)
#pragma unroll
                for (int k = 0; k < 4; ++k) A[i][grp][k] = cb[k];

        __syncthreads();   // the previous item's readers are done with the ring
        const typename Loader::Offsets lofs = Loader::offsets(dw, y0, x0);
        ld.issue_at(src, lofs, z_begin - 1, dd, dh, dw, y0);
        // All fire evaluations of the work item, before the plane loop:
        // evaluation e covers output planes z_begin + e * planes_per_eval onwards.
        for (int e = 0; z_begin + e * planes_per_eval < z_end; ++e) {
            const int zo = z_begin + e * planes_per_eval;
            const int zz = min(zo + (lane >> (lg_opr + 1)), dd - 1);
            const uint64_t row =
                (uint64_t)zz * dh + (uint64_t)(y0 + 2 * wave + ((lane >> lg_opr) & 1));
            const FireBallots fb = fire_ballots(((row * dw + x0) >> 3) + (lane & (opr - 1)), step,
                                                level, batch, seed, threshold);
            uint64_t word = fb.w[0];
#pragma unroll
            for (int b = 1; b < 8; ++b) word = (lane & 7) == b ? fb.w[b] : word;
            fire_words[wave][e][lane & 7] = word;   // 8 lanes per address, same value
        }
        ld.commit(ring[0]);
        ld.issue_at(src, lofs, z_begin, dd, dh, dw, y0);
        __syncthreads();

        // Plane p (j = (p - z_begin + 1) % 3) is in ring slot j, plane p - 1 in
        // slot (j + 2) % 3, and plane p + 1 goes to slot (j + 1) % 3.
        auto body = [&](int p, auto jc) {
            constexpr int j = decltype(jc)::value;
            constexpr int jm = (j + 2) % 3, jp = (j + 1) % 3;
            float (&first)[4][4] = A[jp];    // output p + 1 (dz = -1 weights)
            float (&second)[4][4] = A[j];    // output p (dz = 0)
            float (&last)[4][4] = A[jm];     // output p - 1 (dz = +1), complete after
            const float4 *pl = ring[j];
            // Taps are software-pipelined: the LDS reads of tap t + 1 are issued
            // before the FMAs of tap t, and pinning the sums after each tap keeps
            // the compiler from hoisting every read of the plane at once.
            int gq = g;
            pin(gq);   // re-read the tap weights every plane rather than keep 27 in registers
            float4 sv[2][4], wv[2][3];
            auto read_tap = [&](int t, float4 (&s4)[4], float4 (&w3)[3]) {
                const int off = (t / 3 - 1) * kHaloW + (t % 3 - 1);
                w3[0] = tapw[t][gq];        // dz = -1: output p + 1
                w3[1] = tapw[9 + t][gq];    // dz =  0: output p
                w3[2] = tapw[18 + t][gq];   // dz = +1: output p - 1
#pragma unroll
                for (int grp = 0; grp < 4; ++grp) s4[grp] = pl[centre[grp] + off];
            };
            read_tap(0, sv[0], wv[0]);
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                if (t + 1 < 9) read_tap(t + 1, sv[(t + 1) & 1], wv[(t + 1) & 1]);
                const float4 *w3 = wv[t & 1];
                const float a_m[4] = {w3[0].x, w3[0].y, w3[0].z, w3[0].w};
                const float a_0[4] = {w3[1].x, w3[1].y, w3[1].z, w3[1].w};
                const float a_p[4] = {w3[2].x, w3[2].y, w3[2].z, w3[2].w};
#pragma unroll
                for (int grp = 0; grp < 4; ++grp) {
                    const float4 v = sv[t & 1][grp];
                    const float vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        first[grp][k] = fmaf(a_m[k], vv[k], t == 0 ? cb[k] : first[grp][k]);
                        second[grp][k] = fmaf(a_0[k], vv[k], second[grp][k]);
                        last[grp][k] = fmaf(a_p[k], vv[k], last[grp][k]);
                    }
                }
#pragma unroll
                for (int grp = 0; grp < 4; ++grp)
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        pin(first[grp][k]);
                        pin(second[grp][k]);
                        pin(last[grp][k]);
                    }
            }
            __builtin_amdgcn_sched_barrier(0);

            // output plane zo = p - 1: MLP, fire gate, store (stores of planes
            // outside [z_begin, z_end) are dropped by an empty descriptor)
            const int zo = p - 1;
            const bool out_ok = zo >= z_begin && zo < z_end;
            const int zrel = min(max(zo - z_begin, 0), k3ZRun - 1);   // in range for any plane
            const int phase = zrel & (planes_per_eval - 1);
            const uint64_t *fwe = fire_words[wave][zrel / planes_per_eval];
            const int slot0 = 2 * phase;
            const Rsrc wr = make_rsrc(dst + ((int64_t)max(zo, 0) * dh + y0) * dw * C,
                                      out_ok ? (uint32_t)min(k3TY, dh - y0) * row_bytes : 0u);
            const float4 *own = ring[jm];
            // ALIGNED: the bits of the lane's 4 cells of this plane, at 2 grp
            // (cell n of group grp is cell n % 8 of block 2 (grp % 2) + n / 8
            // of row grp / 2: bit (slot0 + grp / 2) * 4 + 2 (grp % 2) + n / 8)
            uint32_t fw_lane = 0;
            if constexpr (ALIGNED) fw_lane = (uint32_t)(fwe[n & 7] >> (slot0 * opr + (n >> 3)));
#pragma unroll
            for (int grp = 0; grp < 4; ++grp) {
                const float4 sp = own[centre[grp]];
                float f[8] = {sp.x, sp.y, sp.z, sp.w};
#pragma unroll
                for (int k = 0; k < 4; ++k) f[4 + k] = last[grp][k];
                // The MLP of a plane outside the run (the first two bodies of a
                // work item and its padding) is skipped: a uniform branch with
                // no memory operation inside, so the store below and the wait
                // counts around it are the same on both paths.  That store is
                // dropped, so u may hold anything there (left unspecified: no
                // register moves to merge the two paths).
                v4f u = __builtin_nondeterministic_value(u);
                if (out_ok) {
                    v4f acc[4];
                    mlp.layer1(f, acc);
                    u = mlp.layer2(acc);
                }
                float m;
                if constexpr (ALIGNED) {
                    m = (float)__builtin_amdgcn_ubfe(fw_lane, 2u * grp, 1u);
                } else {
                    const int r = grp >> 1;
                    const int y = y0 + 2 * wave + r, x = x0 + (grp & 1) * 16 + n;
                    const uint64_t idx = ((uint64_t)max(zo, 0) * dh + y) * dw + x;
                    const uint64_t row_b0 = (((uint64_t)max(zo, 0) * dh + y) * dw + x0) >> 3;
                    const uint64_t fw = fwe[idx & 7];
                    m = (fw >> ((slot0 + r) * opr + (int)((idx >> 3) - row_b0))) & 1 ? 1.f : 0.f;
                }
                update_store<Mlp>(dst, wr, offs[grp], g, f, u, m);
                __builtin_amdgcn_sched_barrier(0);
            }

            // plane p + 1 into the free slot, then start loading p + 2
            ld.commit(ring[jp]);
            ld.issue_at(src, lofs, p + 2, dd, dh, dw, y0, p + 2 <= z_end);
            __syncthreads();
        };
        for (int p0 = z_begin - 1; p0 <= z_end; p0 += 3) {
            body(p0, std::integral_constant<int, 0>{});
            body(p0 + 1, std::integral_constant<int, 1>{});
            body(p0 + 2, std::integral_constant<int, 2>{});
        }
    }
}

// ==== host side: launch plans and dispatch ====

constexpr int kBlocksPerCu = 2;

// Work layout of a 2D level: row streaming over strips of 32 cells (the 16 x
// 32 tile kernel only when asked for).  A work item is a run of k2RunRows
// rows where the level has at least one such run per SIMD of a full MI355X
// (256 CUs x 4 SIMDs); smaller levels take shorter runs (down to 2 rows) so
// that they still spread over about that many waves: they are bound by the
// latency of a wave's rows, not by throughput, and the extra halo rows of
// short runs cost less than idle SIMDs.  Measured against 16 x 32 tiles:
// medium 2D pass 1.43 -> 1.25 ms, tiny 2D 0.285 -> 0.22 ms, training step
// 3.20 -> 3.07 ms; on those levels one run per wave slot (2 per SIMD) or half a
// run per SIMD was slower.  The row kernel sums the taps in the tile
// kernel's order, so the results are the same bits.  Two steps per launch
// need at least one two-step run per wave slot (kPlanSlots).  Both counts are
// those of a full MI355X, not the device's, so the launch sequence (and with
// it the buffer that holds a result) is the same on every device; only grid
// sizes follow the device.
constexpr int64_t kPlanSlots = 256 * 4 * k2WavesPerSimd;
constexpr int64_t kRowRuns = 256 * 4;

struct RowsPlan {
    int tiles_x;
    int run;                      // rows per work item
    int64_t runs, items, slots;   // slots: wave slots of this device (grid size)
};

// From kLongRun rows a run, more and shorter runs pay: one wave a SIMD leaves
// gaps that its one row in flight does not fill.  Two runs a SIMD do for fp16
// states whose rows start on 8-cell boundaries and for fp32 states whose rows
// do not (their fire draws take twice the lanes); three, the third of which a
// SIMD's waves reach at different times, for fp16 states with such rows; fp32
// states with aligned rows keep one.  Where runs would pass k2RunRows there
// are as many per SIMD as it takes.  A count just above a multiple of the
// SIMDs is the worst case, so runs grow until it is not.  Microseconds a step
// with 1, 2, 3 runs a SIMD: fp16 724^2 19.6, 20.0, 18.1; 999 x 1337 37.7, 33.4,
// 31.3; 1024^2 26.0, 24.0, 25.2; 1408 x 2048 61.7, 50.2, 49.4; fp32 800 x 900
// 25.1, 23.5, 24.7; 999 x 1337 39.7, 38.3, 37.9; 1200 x 1500 51.2, 46.0, 47.6;
// 1024^2 26.7, 29.0, 29.5; 1408 x 2048 74.2, 79.3, 76.2; 600^2 fp16 13.4, 14.1,
// 14.8; 2816 x 2048 in runs of 128 rows (1408) 170 fp32, 127 fp16, with two
// runs a SIMD 153, 103.
constexpr int kLongRun = 17, kLongRunF32 = 20;

RowsPlan rows_plan(const StepArgs &a) {
    RowsPlan r;
    r.tiles_x = (int)((a.ext.w + kTileW - 1) / kTileW);
    r.slots = (int64_t)device_cus() * 4 * k2WavesPerSimd;
    const auto rows = [&](int64_t n) {   // rows of a run with n runs a SIMD
        return std::max<int64_t>(2, (a.ext.h * r.tiles_x + n * kRowRuns - 1) / (n * kRowRuns));
    };
    const bool half = a.dtype == Dtype::F16, aligned = a.ext.w % 8 == 0;
    int64_t run = rows(1);
    if (run >= (half ? kLongRun : kLongRunF32)) {
        int64_t n = 1 + (half ? 1 : 0) + (aligned ? 0 : 1);
        n = std::max(n, (run + k2RunRows - 1) / k2RunRows);
        run = rows(n);
        while (run < k2RunRows && (a.ext.h + run - 1) / run * r.tiles_x > n * kRowRuns) ++run;
    }
    r.run = (int)std::min<int64_t>(k2RunRows, run);
    r.runs = (a.ext.h + r.run - 1) / r.run;
    r.items = (int64_t)r.tiles_x * r.runs;
    return r;
}

bool uses_rows(const StepArgs &, Layout2d layout) { return layout != Layout2d::Tiles; }

// Row kernel launch; UP: the first step of a level fused with the upsample
// from the coarse state src (width cdw) by (fy, fx) and the image img.
template <typename T, int NIN, class Mlp, bool UP>
hipError_t launch_rows(const StepArgs &a, const void *src, void *dst, const void *img, int cdw,
                       int fy, int fx, hipStream_t stream) {
    const RowsPlan r = rows_plan(a);
    if (r.items == 0) return hipSuccess;
    if (r.items > INT32_MAX) return hipErrorInvalidValue;
    const int grid = (int)std::min<int64_t>(r.items, r.slots);
    auto kern = a.ext.w % 8 == 0 ? nca_step_mfma_2d_rows<T, NIN, Mlp, true, UP>
                                 : nca_step_mfma_2d_rows<T, NIN, Mlp, false, UP>;
    kern<<<grid, 64, 0, stream>>>(
        (const T *)src, (T *)dst, (int)a.ext.h, (int)a.ext.w, r.tiles_x, (int)r.runs, r.run,
        (int)r.items, a.w.conv_w, a.w.conv_b, a.w.w1, a.w.b1, a.w.w2, a.level, a.step, a.batch,
        a.seed, a.threshold, (const T *)img, cdw, fy, fx);
    return hipGetLastError();
}

// Two-step row kernel: strips of 30 output cells; used where the single-step
// kernel would use the row layout (fp32 states, default MLP).
RowsPlan pair_plan(const StepArgs &a) {
    RowsPlan r;
    r.tiles_x = (int)((a.ext.w + k2PairW - 1) / k2PairW);
    r.slots = (int64_t)device_cus() * 4 * k2WavesPerSimd;
    r.runs = (a.ext.h + k2RunRows - 1) / k2RunRows;
    r.items = (int64_t)r.tiles_x * r.runs;
    return r;
}

// The ablation's C = 12, H = 48 model (supplement S10) on the kernels of
// C = 16: the 2D row kernels and the 3D step with an fp32 ring, the default
// operands, the lanes of channel quad 3 and hidden tile 3 idle.  (fp16 3D: the
// step of C = 16 rounds taps and perception to fp16, which these steps never
// did.  With the fp32 ring the finest level's step of a 48 x 120 x 216 clip
// takes 47 us, on the generic kernel 105.)
using MlpC12 = MlpF16SM<12, 48>;
using MlpC12h = MlpF16M<12, 48>;
bool is_c12(const StepArgs &a) { return a.channels == 12 && a.hidden == 48; }
bool is_c16(const StepArgs &a) { return a.channels == kC && a.hidden == kH; }

bool uses_pairs(const StepArgs &a, MfmaMlp mlp, Layout2d layout) {
    return a.ndim == 2 && a.dtype == Dtype::F32 && (is_c16(a) || is_c12(a)) &&
           a.ext.h * a.ext.w < (int64_t(1) << 32) &&   // 32-bit cell indices in the kernel
           (mlp == MfmaMlp::Default || mlp == MfmaMlp::F16S) &&
           (layout == Layout2d::Rows ||
            (layout == Layout2d::Auto && pair_plan(a).items >= kPlanSlots));
}

// UP: src is the coarse state (width cdw) upsampled by (fy, fx), img the
// level's image; steps a.step and a.step + 1.
template <class Mlp, int NIN, bool UP>
hipError_t launch_rows_pair(const StepArgs &a, const void *src, void *dst, const void *img,
                            int cdw, int fy, int fx, hipStream_t stream) {
    const RowsPlan r = pair_plan(a);
    if (r.items == 0) return hipSuccess;
    if (r.items > INT32_MAX) return hipErrorInvalidValue;
    const int grid = (int)std::min<int64_t>(r.items, r.slots);
    auto kern = a.seg != nullptr ? nca_step2_mfma_2d_rows<float, NIN, Mlp, UP, true>
                                 : nca_step2_mfma_2d_rows<float, NIN, Mlp, UP, false>;
    kern<<<grid, 64, 0, stream>>>(
        (const float *)src, (float *)dst, (int)a.ext.h, (int)a.ext.w, r.tiles_x, k2RunRows,
        (int)r.items, a.w.conv_w, a.w.conv_b, a.w.w1, a.w.b1, a.w.w2, a.level, a.step, a.batch,
        a.seed, a.threshold, (const float *)img, cdw, fy, fx, a.seg);
    return hipGetLastError();
}

template <typename T, int NIN, class Mlp>
hipError_t launch_2d(const StepArgs &a, Layout2d layout, const void *src, void *dst,
                     hipStream_t stream) {
    const int tiles_x = (int)((a.ext.w + kTileW - 1) / kTileW);
    const int tiles_y = (int)((a.ext.h + k2TY - 1) / k2TY);
    const int64_t tiles = (int64_t)tiles_x * tiles_y;
    if (tiles == 0) return hipSuccess;
    if (tiles > INT32_MAX) return hipErrorInvalidValue;
    if (uses_rows(a, layout))
        return launch_rows<T, NIN, Mlp, false>(a, src, dst, nullptr, 0, 1, 1, stream);
    if constexpr (Mlp::kChannels != kC) {
        return hipErrorInvalidValue;   // other model sizes: rows only
    } else {
        const int grid = (int)std::min<int64_t>(tiles, (int64_t)device_cus() * k2BlocksPerCu);
        nca_step_mfma_2d<T, NIN, Mlp><<<grid, kThreads, 0, stream>>>(
            (const T *)src, (T *)dst, (int)a.ext.h, (int)a.ext.w, tiles_x, (int)tiles,
            a.w.conv_w, a.w.conv_b, a.w.w1, a.w.b1, a.w.w2, a.level, a.step, a.batch, a.seed,
            a.threshold);
        return hipGetLastError();
    }
}

template <typename T, int NIN, class Mlp>
hipError_t launch_3d(const StepArgs &a, const void *src, void *dst, hipStream_t stream) {
    if constexpr (std::is_same_v<T, __half> && std::is_same_v<Mlp, MlpF16>) {
        return launch_step_3d_f16(a, src, dst, nullptr, 0, 0, 1, 1, 1, stream);
    } else {
        const int tiles_x = (int)((a.ext.w + kTileW - 1) / kTileW);
        const int tiles_y = (int)((a.ext.h + k3TY - 1) / k3TY);
        const int64_t slots = (int64_t)device_cus() * kBlocksPerCu;
        const int zrun = pick_zrun((int64_t)tiles_x * tiles_y, a.ext.d, slots, k3ZRun);
        const int64_t zruns = (a.ext.d + zrun - 1) / zrun;
        const int64_t items = (int64_t)tiles_x * tiles_y * zruns;
        if (items == 0) return hipSuccess;
        if (items > INT32_MAX) return hipErrorInvalidValue;
        const int grid = (int)std::min<int64_t>(items, slots);
        auto kern = a.ext.w % 8 == 0 ? nca_step_mfma_3d<T, NIN, Mlp, true>
                                     : nca_step_mfma_3d<T, NIN, Mlp, false>;
        kern<<<grid, kThreads, 0, stream>>>(
            (const T *)src, (T *)dst, (int)a.ext.d, (int)a.ext.h, (int)a.ext.w, tiles_x, tiles_y,
            (int)items, zrun, a.w.conv_w, a.w.conv_b, a.w.w1, a.w.b1, a.w.w2, a.level, a.step,
            a.batch, a.seed, a.threshold);
        return hipGetLastError();
    }
}

template <typename T, class Mlp>
hipError_t dispatch(const StepArgs &a, Layout2d layout, const void *src, void *dst,
                    hipStream_t stream) {
    if (a.ndim == 2) {
        if (a.n_in == 1) return launch_2d<T, 1, Mlp>(a, layout, src, dst, stream);
        if (a.n_in == 3) return launch_2d<T, 3, Mlp>(a, layout, src, dst, stream);
    } else {
        if (a.n_in == 1) return launch_3d<T, 1, Mlp>(a, src, dst, stream);
        if (a.n_in == 3) return launch_3d<T, 3, Mlp>(a, src, dst, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace

bool mfma_fits(const StepArgs &a) {
    // Buffer descriptors address a tile's rows with 32-bit offsets: rows of
    // more than (2^32 / 18 rows) bytes go to the vector kernel instead.
    const int64_t cell_bytes = (int64_t)kC * (a.dtype == Dtype::F32 ? 4 : 2);
    return (int64_t)(k2TY + 2) * a.ext.w * cell_bytes < (int64_t(1) << 32);
}

bool step_mfma_single_readout(const StepArgs &a, MfmaMlp mlp) {
    return a.ndim == 3 && a.dtype == Dtype::F16 && a.channels == kC && a.hidden == kH &&
           (mlp == MfmaMlp::Default || mlp == MfmaMlp::F16) && mfma_fits(a);
}

bool step_mfma_pairs(const StepArgs &a, MfmaMlp mlp, Layout2d layout) {
    return mfma_fits(a) && uses_pairs(a, mlp, layout);
}

template <class Mlp>
hipError_t launch_pair_size(const StepArgs &a, const void *src, void *dst, const void *img,
                            int cdw, int fy, int fx, bool up, hipStream_t stream) {
    if (a.n_in == 1)
        return up ? launch_rows_pair<Mlp, 1, true>(a, src, dst, img, cdw, fy, fx, stream)
                  : launch_rows_pair<Mlp, 1, false>(a, src, dst, nullptr, 0, 1, 1, stream);
    if (a.n_in == 3)
        return up ? launch_rows_pair<Mlp, 3, true>(a, src, dst, img, cdw, fy, fx, stream)
                  : launch_rows_pair<Mlp, 3, false>(a, src, dst, nullptr, 0, 1, 1, stream);
    return hipErrorInvalidValue;
}

hipError_t launch_step2_mfma(const StepArgs &a, MfmaMlp mlp, Layout2d layout, const void *src,
                             void *dst, hipStream_t stream) {
    if (!step_mfma_pairs(a, mlp, layout)) return hipErrorInvalidValue;
    return is_c12(a) ? launch_pair_size<MlpC12>(a, src, dst, nullptr, 0, 1, 1, false, stream)
                     : launch_pair_size<MlpF32State>(a, src, dst, nullptr, 0, 1, 1, false, stream);
}

hipError_t launch_step2_mfma_up(const StepArgs &a, MfmaMlp mlp, Layout2d layout,
                                const void *coarse, int coarse_w, int fy, int fx, const void *img,
                                void *dst, hipStream_t stream) {
    if (!step_mfma_pairs(a, mlp, layout)) return hipErrorInvalidValue;
    return is_c12(a)
               ? launch_pair_size<MlpC12>(a, coarse, dst, img, coarse_w, fy, fx, true, stream)
               : launch_pair_size<MlpF32State>(a, coarse, dst, img, coarse_w, fy, fx, true, stream);
}

// fp16 volumes of two planes of the 12 / 48 model stay on the generic kernel from
// this many cells a plane on: its tiles are two planes, where a run of the 3D step
// streams four or six for them.  Generic kernel and 3D step, us a step: 2 x 160 x
// 160 cells 11.3, 10.5; 200^2 12.9, 13.4; 250^2 12.8, 14.6; 300^2 19.7, 21.8; 350 x
// 400 27.6, 32.5; 800^2 83, 88; 1000 x 1500 182, 235.  One plane of 300^2 17.7,
// 13.6, three 31.5, 22.7, four of 200^2 21.4, 17.1.
constexpr int64_t kTwoPlanes = 32000;

bool step_mfma_serves(const StepArgs &a, Layout2d layout) {
    if (is_c16(a)) return true;
    if (a.ndim == 3 && a.dtype == Dtype::F16 && a.ext.d == 2 && a.ext.h * a.ext.w >= kTwoPlanes)
        return false;
    return is_c12(a) && (a.ndim == 3 || uses_rows(a, layout)) && mfma_fits(a);
}

bool step_mfma_fuses_upsample(const StepArgs &a, MfmaMlp mlp, Layout2d layout) {
    if (mlp != MfmaMlp::Default || !mfma_fits(a)) return false;
    if (is_c12(a)) return a.ndim == 2 && step_mfma_serves(a, layout);
    if (!is_c16(a)) return false;
    if (a.ndim == 2) return uses_rows(a, layout);
    return a.dtype == Dtype::F16;   // the fp16 3D step
}

hipError_t launch_step_mfma_up(const StepArgs &a, Layout2d layout, const void *coarse,
                               int coarse_h, int coarse_w, int fz, int fy, int fx,
                               const void *img, void *dst, hipStream_t stream) {
    if (!step_mfma_fuses_upsample(a, MfmaMlp::Default, layout)) return hipErrorInvalidValue;
    if (a.ndim == 3)
        return launch_step_3d_f16(a, coarse, dst, img, coarse_h, coarse_w, fz, fy, fx, stream);
    if (is_c12(a) && a.dtype == Dtype::F16) {
        if (a.n_in == 1)
            return launch_rows<__half, 1, MlpC12h, true>(a, coarse, dst, img, coarse_w, fy, fx,
                                                         stream);
        if (a.n_in == 3)
            return launch_rows<__half, 3, MlpC12h, true>(a, coarse, dst, img, coarse_w, fy, fx,
                                                         stream);
        return hipErrorInvalidValue;
    }
    if (is_c12(a)) {
        if (a.n_in == 1)
            return launch_rows<float, 1, MlpC12, true>(a, coarse, dst, img, coarse_w, fy, fx,
                                                       stream);
        if (a.n_in == 3)
            return launch_rows<float, 3, MlpC12, true>(a, coarse, dst, img, coarse_w, fy, fx,
                                                       stream);
        return hipErrorInvalidValue;
    }
    if (a.dtype == Dtype::F32) {
        if (a.n_in == 1)
            return launch_rows<float, 1, MlpF32State, true>(a, coarse, dst, img, coarse_w, fy, fx,
                                                            stream);
        if (a.n_in == 3)
            return launch_rows<float, 3, MlpF32State, true>(a, coarse, dst, img, coarse_w, fy, fx,
                                                            stream);
    } else {
        if (a.n_in == 1)
            return launch_rows<__half, 1, MlpF16, true>(a, coarse, dst, img, coarse_w, fy, fx,
                                                        stream);
        if (a.n_in == 3)
            return launch_rows<__half, 3, MlpF16, true>(a, coarse, dst, img, coarse_w, fy, fx,
                                                        stream);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_step_mfma(const StepArgs &a, MfmaMlp mlp, Layout2d layout, const void *src,
                            void *dst, hipStream_t stream) {
    if (!mfma_fits(a)) return launch_step_valu(a, src, dst, stream);
    if (is_c12(a)) {
        if (!step_mfma_serves(a, layout) || mlp != MfmaMlp::Default) return hipErrorInvalidValue;
        return a.dtype == Dtype::F32 ? dispatch<float, MlpC12>(a, layout, src, dst, stream)
                                     : dispatch<__half, MlpC12h>(a, layout, src, dst, stream);
    }
    if (!is_c16(a)) return hipErrorInvalidValue;
    if (mlp == MfmaMlp::Default)
        mlp = a.dtype == Dtype::F32 ? MfmaMlp::F16S : MfmaMlp::F16;
    if (a.dtype == Dtype::F32) {
        switch (mlp) {
            case MfmaMlp::F32: return dispatch<float, MlpF32>(a, layout, src, dst, stream);
            case MfmaMlp::Bf16x3: return dispatch<float, MlpBf16x3>(a, layout, src, dst, stream);
            case MfmaMlp::F16S: return dispatch<float, MlpF32State>(a, layout, src, dst, stream);
            default: return hipErrorInvalidValue;   // fp16 operands are too coarse for fp32 states
        }
    }
    switch (mlp) {
        case MfmaMlp::F32: return dispatch<__half, MlpF32>(a, layout, src, dst, stream);
        case MfmaMlp::Bf16x3: return dispatch<__half, MlpBf16x3>(a, layout, src, dst, stream);
        case MfmaMlp::F16: return dispatch<__half, MlpF16>(a, layout, src, dst, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace octnca
