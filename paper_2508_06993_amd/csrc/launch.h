// Internal launch interface between the C ABI layer (api.hip) and the kernel
// files.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>

#include "device_common.h"

namespace octnca {

struct Extent3 {
    int64_t d, h, w;
    int64_t cells() const { return d * h * w; }
};

enum class Dtype : int { F32 = 0, F16 = 1 };

// Pyramid: dst = mean of src over (fz, fy, fx) blocks; dst_ext = src_ext / f.
hipError_t launch_pool(Dtype dt, const void *src, Extent3 dst_ext, void *dst, int fz, int fy,
                       int fx, int n_in, hipStream_t stream);

// Upsample + inject.  coarse == nullptr seeds the hidden channels with zeros
// (coarsest level initialisation, factors then must be 1).
hipError_t launch_upsample(Dtype dt, const void *coarse, Extent3 fine_ext, int fz, int fy, int fx,
                           const void *img, void *fine, int n_in, int channels,
                           hipStream_t stream);
hipError_t launch_readout(Dtype dt, const void *state, int64_t cells, int channels, uint8_t *seg,
                          hipStream_t stream);
hipError_t launch_readout_classes(Dtype dt, const void *state, int64_t cells, int channels,
                                  int classes, uint8_t *seg, hipStream_t stream);

hipError_t launch_fire_mask(uint64_t seed, uint32_t level, uint32_t step, int64_t cells,
                            uint64_t threshold, uint8_t *mask, hipStream_t stream);

// MLP operand precision of the MFMA step kernel.  Default: scaled fp16
// activations with split fp16 weights (F16S) for fp32 states, fp16 for fp16 states.
enum class MfmaMlp : int { Default = 0, F32 = 1, Bf16x3 = 2, F16 = 3, F16S = 4 };
// Work layout of the 2D MFMA step.  Auto: row streaming on large levels,
// 16 x 32 tiles on small ones; Rows / Tiles force one (3D steps ignore it).
enum class Layout2d : int { Auto = 0, Rows = 1, Tiles = 2 };
// Step kernel chosen by the caller (the model description of the C ABI):
// vector kernel or matrix cores, MLP operands, 2D work layout, and whether
// two steps may run in one launch.  The default-constructed value is the
// library's default.
struct KernelChoice {
    bool valu = false;    // one thread per cell on the vector ALUs
    bool pairs = true;    // two steps per launch where the two-step kernel applies
    MfmaMlp mlp = MfmaMlp::Default;
    Layout2d layout = Layout2d::Auto;
};

// One NCA step src -> dst over a level of extent `ext`.
struct StepArgs {
    Dtype dtype;
    int ndim;
    int n_in;
    Extent3 ext;
    LevelWeightsDev w;
    uint32_t level;
    uint32_t step;
    uint32_t batch = 0;   // image index in a batch (fire-mask counter word 3)
    int channels = kC;    // C and H of the model (the matrix-core kernels need 16 / 64)
    int hidden = kH;
    uint64_t seed;
    uint64_t threshold;
    // Device [cells] uint8 or null: a two-step launch, or a single fp16 3D
    // step (see step_single_fuses_readout), also writes the
    // two-class readout of the state it stores.
    uint8_t *seg = nullptr;
    KernelChoice kc;      // step kernel of the matrix-core / vector paths
};
hipError_t launch_step(const StepArgs &a, const void *src, void *dst, hipStream_t stream);
// Whether launch_step would fuse a level's first step with the upsample from
// the next coarser level (see launch_step_mfma_up), and that fused launch.
bool step_fuses_upsample(const StepArgs &a);
hipError_t launch_step_up(const StepArgs &a, const void *coarse, int coarse_h, int coarse_w,
                          int fz, int fy, int fx, const void *img, void *dst,
                          hipStream_t stream);
hipError_t launch_step_valu(const StepArgs &a, const void *src, void *dst, hipStream_t stream);
// Generic matrix-core step for the model sizes other than C = 16, H = 64 (the
// ablation's 12 / 48, where the specialised steps do not run it, and 20 / 100):
// whether it serves `a`, and the launch.
bool step_gen_serves(const StepArgs &a);
hipError_t launch_step_gen(const StepArgs &a, const void *src, void *dst, hipStream_t stream);
// Whether launch_step_pair runs steps a.step and a.step + 1 in one launch, and
// that launch (the state after step a.step is not written to memory).
bool step_pairs(const StepArgs &a);
// Whether the single-step launch that launch_step makes for `a` writes StepArgs::seg.
bool step_single_fuses_readout(const StepArgs &a);
hipError_t launch_step_pair(const StepArgs &a, const void *src, void *dst, hipStream_t stream);
// The first two steps of a level, the first fused with the upsample (when
// step_pairs and step_fuses_upsample both hold).
hipError_t launch_step_pair_up(const StepArgs &a, const void *coarse, int coarse_w, int fz,
                               int fy, int fx, const void *img, void *dst, hipStream_t stream);

// Several steps of a small 2D level in one launch (step_block.hip).
// step_block_plan: whether a run of `steps` steps (of `images` images at once)
// takes these launches, and how: `launches` of them, launch i running
// steps / launches steps, one more for i < steps % launches, on tiles of
// `tile` x `tile` cells.  tape: the training forward (split-bf16 operands).
// same_parity: only plans whose number of launches is odd where `steps` is (for
// a caller whose result has to be in one of two buffers).
struct StepBlockPlan {
    int tile = 0;
    int launches = 0;
    double us = 0;   // the model's time, of these launches or of one per step where those win
    int steps_of(int i, int steps) const { return steps / launches + (i < steps % launches); }
};
bool step_block_plan(const StepArgs &a, bool tape, int steps, int images, StepBlockPlan *plan,
                     bool same_parity = false);
// Where a launch's first state comes from: img null, a state of the level at
// src; else the coarse state at src (width coarse_w, factors fy, fx) with the
// level's image, or with src null the image and zero hidden channels.
// Strides (elements) between the images of a batch.
struct StepBlockInput {
    const void *img = nullptr;
    int coarse_w = 0, fy = 1, fx = 1;
    int images = 1;
    int64_t src_stride = 0, dst_stride = 0, img_stride = 0;
};
// Steps a.step .. a.step + steps - 1; dst receives the last state, or with
// `tape` the state after step a.step + s at dst + s states.  a.seg: readout of
// the last state, or null.
hipError_t launch_step_block(const StepArgs &a, bool tape, int tile, int steps, const void *src,
                             void *dst, StepBlockInput in, hipStream_t stream);

// Training (fp32 states): backward of one step (state `src` before the step,
// gout = dL/dS'), writing gin = dL/dS (may alias gout) and adding the weight
// gradients to g; ws holds step_backward_workspace_floats floats.
size_t step_backward_workspace_floats(int ndim, int channels, int hidden, Extent3 extent);
hipError_t launch_step_backward(const StepArgs &a, const float *src, const float *gout,
                                float *gin, LevelGradsDev g, float *ws, hipStream_t stream);
// Backward of all `steps` steps of a level (a.step unused): states holds the
// level's states before steps 0 .. steps-1 (state t at states + t * cells * C),
// gout = dL/dS after the last step; gin receives dL/dS of the level's first
// state (must not alias gout or states) and g receives the level's weight
// gradients (written, not added: the buffers need no clearing).  ws holds
// level_backward_workspace_floats floats.  steps = 0 enqueues nothing (neither
// gin nor g is written).
size_t level_backward_workspace_floats(int ndim, int channels, int hidden, Extent3 extent);
hipError_t launch_level_backward(const StepArgs &a, int32_t steps, const float *states,
                                 const float *gout, float *gin, LevelGradsDev g, float *ws,
                                 hipStream_t stream);
// The backward's per-cell part on large tiles (bwd_block.hip; C = 16, H = 64):
// whether it runs a level of `steps` steps, and how: `launches` launches,
// launch i running steps / launches steps, one more for i < steps % launches,
// on tiles of `tile` x `tile` cells (2D; 4 x 8 x 8 and one step in 3D), each
// block with a row of weight-gradient sums (bwd_block_rows of them, at most
// max_blocks).
struct BwdBlockPlan {
    int tile = 0;
    int launches = 0;
    int steps_of(int i, int steps) const { return steps / launches + (i < steps % launches); }
};
bool bwd_block_plan(const StepArgs &a, int steps, int64_t max_blocks, BwdBlockPlan *plan);
int64_t bwd_block_rows(const StepArgs &a, const BwdBlockPlan &plan);
// Backward of steps a.step, a.step - 1, .. (steps of them): state is the state
// before step a.step, the earlier ones lie one state of the level before it
// each.  G' = gout + conv^T(gp_prev) (gp_prev null: gout); gpart and gp
// receive G' + gS and gP of the last of these steps, both [cells][C].
hipError_t launch_bwd_block(const StepArgs &a, const BwdBlockPlan &plan, int steps,
                            const float *state, const float *gout, const float *gp_prev,
                            float *gpart, float *gp, float *partial, bool accumulate,
                            hipStream_t stream);
// Adjoint of the upsample + inject from `coarse` (extent of the coarse level).
hipError_t launch_upsample_adjoint(const float *gfine, Extent3 coarse, int fz, int fy, int fx,
                                   int n_in, int channels, float *gcoarse, hipStream_t stream);
// Readout-channel MSE: grad = dL/dS, *loss = L (device); ws holds
// mse_workspace_doubles doubles.
size_t mse_workspace_doubles(int64_t cells);
hipError_t launch_readout_mse(const float *state, const float *target, int64_t cells, int channels,
                              float *grad, double *loss, double *ws, hipStream_t stream);
hipError_t launch_fill_zero(float *p, int64_t n, hipStream_t stream);
// The specialised matrix-core steps: every step of C = 16, H = 64 models and,
// with the default operand policy, of C = 12, H = 48 models the 2D steps in the
// row layout and the 3D ones (but fp16 volumes of two large planes);
// step_mfma_serves says whether launch_step_mfma runs `a`.
bool step_mfma_serves(const StepArgs &a, Layout2d layout);
hipError_t launch_step_mfma(const StepArgs &a, MfmaMlp mlp, Layout2d layout, const void *src,
                            void *dst, hipStream_t stream);
// The first step of a level fused with the upsample + inject from the next
// coarser level (2D row-streaming kernel and fp16 3D step, default operand
// policy only):
// step_mfma_fuses_upsample says whether launch_step_mfma would run that kernel
// for `a`; launch_step_mfma_up then reads the coarse state (width coarse_w,
// factors fy, fx) and the level's image instead of a state of the level.
bool step_mfma_fuses_upsample(const StepArgs &a, MfmaMlp mlp, Layout2d layout);
// Two steps, a.step and a.step + 1, in one launch (2D fp32 row layout, default
// operand policy): step_mfma_pairs says whether that kernel exists for `a`;
// launch_step2_mfma reads src and writes the state after both steps to dst.
bool step_mfma_pairs(const StepArgs &a, MfmaMlp mlp, Layout2d layout);
// Whether a single-step launch of launch_step_mfma for `a` writes StepArgs::seg.
bool step_mfma_single_readout(const StepArgs &a, MfmaMlp mlp);
hipError_t launch_step2_mfma(const StepArgs &a, MfmaMlp mlp, Layout2d layout, const void *src,
                             void *dst, hipStream_t stream);
// The same two steps with step a.step fused with the upsample + inject from
// the coarse state (width coarse_w, factors fy, fx) and the level's image.
hipError_t launch_step2_mfma_up(const StepArgs &a, MfmaMlp mlp, Layout2d layout,
                                const void *coarse, int coarse_w, int fy, int fx, const void *img,
                                void *dst, hipStream_t stream);
hipError_t launch_step_mfma_up(const StepArgs &a, Layout2d layout, const void *coarse,
                               int coarse_h, int coarse_w, int fz, int fy, int fx,
                               const void *img, void *dst, hipStream_t stream);

// Compute units of the current device, cached per device.  Host threads may
// call this concurrently: racing first calls store the same value.
inline int device_cus() {
    static std::atomic<int> cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            n <= 0)
            n = 256;
        cached[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

// Output planes per work item of the fp32-ring 3D step, chosen per launch: the
// run length r in 1 .. max_run that minimises ceil(items(r) / slots) *
// (min(r, depth) + 2, rounded up to whole groups of three), the work of the
// most loaded block slot (grid-stride rounds times the planes a work item
// streams, its halo planes included; the plane loop is unrolled three times);
// ties go to the longer run.  Short runs spread small levels over the chip at
// the cost of reading their halo planes again; long runs stream large levels
// with little re-reading.
inline int pick_zrun(int64_t tiles, int64_t depth, int64_t slots, int max_run) {
    int best = 1;
    int64_t best_cost = INT64_MAX;
    for (int r = 1; r <= max_run; ++r) {
        const int64_t items = tiles * ((depth + r - 1) / r);
        const int64_t planes = (std::min<int64_t>(r, depth) + 4) / 3 * 3;
        const int64_t cost = (items + slots - 1) / slots * planes;
        if (cost <= best_cost) {
            best_cost = cost;
            best = r;
        }
    }
    return best;
}

// The fp16 3D step of C = 16, H = 64 models with fp16 MLP operands
// (step_3d_f16.hip); img null: src is a state of the level, else the first step
// fused with the upsample from the coarse state src (planes of cdh x cdw cells).
hipError_t launch_step_3d_f16(const StepArgs &a, const void *src, void *dst, const void *img,
                              int cdh, int cdw, int fz, int fy, int fx, hipStream_t stream);
// Its run length (planes per work item, at most max_run) for a level of `depth`
// planes of `tiles` tiles on a device of `cus` CUs.
int step_3d_f16_run(int64_t tiles, int64_t depth, int64_t cus, int max_run);

}  // namespace octnca
