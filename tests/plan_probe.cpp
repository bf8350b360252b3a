// Prints the launch plans of the library's host code, one line per query read
// from stdin, for the tests of the plans.
//   block <dtype> <c> <h> <rows> <cols> <steps> <images> <same_parity> -> use tile launches
//   bwd <ndim> <d> <rows> <cols> <steps> -> use tile launches rows (of gradient sums)
//   serves <dtype> <c> <h> <d> <rows> <cols> -> whether the specialised kernels run a 3D step
//   run <d> <rows> <cols> -> planes of a work item of the fp16 3D step (256 CUs)
#include <cstdio>
#include <cstring>

#include "launch.h"

using namespace octnca;

namespace {

StepArgs args(const char *dtype, int ndim, int c, int h, long d, long rows, long cols) {
    StepArgs a{};
    a.dtype = std::strcmp(dtype, "f16") ? Dtype::F32 : Dtype::F16;
    a.ndim = ndim;
    a.n_in = 3;
    a.ext = Extent3{d, rows, cols};
    a.channels = c;
    a.hidden = h;
    return a;
}

}  // namespace

int main() {
    char what[16], dtype[8];
    while (std::scanf("%15s", what) == 1) {
        if (!std::strcmp(what, "block")) {
            int c, h, steps, images, parity;
            long rows, cols;
            if (std::scanf("%7s %d %d %ld %ld %d %d %d", dtype, &c, &h, &rows, &cols, &steps,
                           &images, &parity) != 8)
                return 1;
            StepBlockPlan p;
            const bool use = step_block_plan(args(dtype, 2, c, h, 1, rows, cols), false, steps,
                                             images, &p, parity != 0);
            std::printf("%d %d %d\n", use ? 1 : 0, use ? p.tile : 0, use ? p.launches : 0);
        } else if (!std::strcmp(what, "bwd")) {
            int ndim, steps;
            long d, rows, cols;
            if (std::scanf("%d %ld %ld %ld %d", &ndim, &d, &rows, &cols, &steps) != 5) return 1;
            BwdBlockPlan p;
            const bool use = bwd_block_plan(args("f32", ndim, 16, 64, d, rows, cols), steps,
                                            int64_t(1) << 30, &p);
            const StepArgs a = args("f32", ndim, 16, 64, d, rows, cols);
            std::printf("%d %d %d %lld\n", use ? 1 : 0, use ? p.tile : 0, use ? p.launches : 0,
                        use ? (long long)bwd_block_rows(a, p) : 0ll);
        } else if (!std::strcmp(what, "serves")) {
            int c, h;
            long d, rows, cols;
            if (std::scanf("%7s %d %d %ld %ld %ld", dtype, &c, &h, &d, &rows, &cols) != 6) return 1;
            const StepArgs a = args(dtype, 3, c, h, d, rows, cols);
            std::printf("%d\n", step_mfma_serves(a, Layout2d::Auto) ? 1 : 0);
        } else if (!std::strcmp(what, "run")) {
            long d, rows, cols;
            if (std::scanf("%ld %ld %ld", &d, &rows, &cols) != 3) return 1;
            std::printf("%d\n", step_3d_f16_run((rows + 7) / 8 * ((cols + 31) / 32), d, 256,
                                                cols % 8 == 0 ? 256 : 128));
        } else {
            return 1;
        }
    }
    return 0;
}
