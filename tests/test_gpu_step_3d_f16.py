"""The fp16 3D step's perception on the matrix cores (step_3d_f16.hip): one
step and several against the vector kernel, whose perception sums the same
fp16 states and fp32 taps one by one in fp32, at sizes around its 8 x 32 tiles
and 2 x 8 blocks, with runs of one and two planes and (48 x 120 x 216, 60 x 108 x 212,
300 x 40 x 64) of 6 and 12; and cells that are not finite, which must reach their
own 3 x 3 x 3 neighbours only, with the values that the vector kernel gives, in
the plain step and in those fused with the upsample and the readout.

Bound: one step rounds taps, perception, features and hidden units to fp16
(2^-11 each) and stores fp16; sums of 27 and 32 products of N(0, 1) states keep
the relative error of the largest value below 8 * 2^-11 = 4e-3 (five steps:
sqrt(5) times that, below 1e-2)."""
import pytest
import torch

import paper_2508_06993_amd as octnca
from paper_2508_06993_amd.runtime import Inference, upload_weights
from synthetic import VIDEO_2DT, make_weights, scaled

pytestmark = pytest.mark.gpu


def _run(kernel, state, weights, n_in, steps, rate=0.5):
    model = octnca.Model(ndim=3, n_in=n_in, dtype="f16", kernel=kernel)
    b0, b1 = state.clone(), torch.full_like(state, float("nan"))
    at = octnca.octree_nca_run_level(model, b0, b1, weights, 1, steps, rate, 1234)
    torch.cuda.synchronize()
    return b1 if at else b0


def _setup(shape, n_in, seed=3):
    wl = scaled(VIDEO_2DT, shape, n_in=n_in, factors=(), steps=(1,))
    weights = upload_weights(make_weights(wl, seed))[0]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return weights, torch.randn(shape + (16,), generator=gen, device="cuda").half()


@pytest.mark.parametrize("n_in", [1, 3])
@pytest.mark.parametrize("shape", [(1, 1, 1), (2, 8, 32), (3, 9, 33), (5, 7, 31), (1, 40, 8),
                                   (7, 17, 66), (300, 3, 5), (37, 24, 100), (4, 10, 34),
                                   (300, 40, 64), (48, 120, 216), (60, 108, 212)])
@pytest.mark.parametrize("steps", [1, 5])
def test_steps_match_vector_kernel(shape, n_in, steps):
    weights, state = _setup(shape, n_in)
    got = _run("mfma", state, weights, n_in, steps).float()
    want = _run("valu", state, weights, n_in, steps).float()
    assert torch.isfinite(got).all()
    tol = 4e-3 if steps == 1 else 1e-2
    assert float((got - want).abs().max()) <= tol * max(1.0, float(want.abs().max()))
    assert torch.equal(got[..., :n_in], state.float()[..., :n_in])


def _kinds(t):
    """0 finite, 1 / -1 infinite, 2 NaN."""
    t = t.float()
    return torch.where(t.isnan(), 2.0, torch.where(t.isinf(), t.sign(), 0.0))


# spots at corners, on tile, block and fire-byte edges and inside them, in the
# first, a middle and the last plane of a run (runs of 1 and of 12 planes)
SPOTS = {
    (6, 21, 70): [(0, 0, 0), (3, 10, 33), (5, 20, 69), (2, 4, 8)],
    (48, 120, 216): [(0, 0, 0), (11, 7, 31), (12, 60, 101), (17, 8, 32), (18, 33, 7), (30, 119, 215),
                     (47, 100, 150)],
    (60, 108, 212): [(0, 107, 211), (5, 9, 35), (11, 50, 64), (24, 51, 131), (35, 0, 100), (59, 64, 3)],
}


@pytest.mark.parametrize("shape", list(SPOTS))
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
def test_values_that_are_not_finite_stay_local(shape, value):
    n_in = 3
    weights, state = _setup(shape, n_in)
    weights["conv_w"][5, 13] = 0.0       # 0 * infinity: a tap, not a cell outside the stencil
    clean = _run("mfma", state, weights, n_in, 1, rate=1.0).float()
    near = torch.zeros(shape, dtype=torch.bool, device="cuda")
    dirty = state.clone()
    for i, (z, y, x) in enumerate(SPOTS[shape]):
        dirty[z, y, x, (7, 5, 12)[i % 3]] = value
        near[max(0, z - 1):z + 2, max(0, y - 1):y + 2, max(0, x - 1):x + 2] = True
    got = _run("mfma", dirty, weights, n_in, 1, rate=1.0).float()
    assert torch.isfinite(got[~near]).all()
    assert float((got - clean)[~near].abs().max()) <= 4e-3 * float(clean.abs().max())
    # the same hidden channels are infinite or NaN as by the vector kernel (it
    # writes no update to the input channels; here 0 * infinity may reach them)
    want = _run("valu", dirty, weights, n_in, 1, rate=1.0).float()
    assert torch.equal(_kinds(got)[..., n_in:], _kinds(want)[..., n_in:])
    ok = torch.isfinite(want) & torch.isfinite(got)
    assert float((got - want)[ok].abs().max()) <= 4e-3 * float(clean.abs().max())


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("extent,factor", [((6, 20, 70), (1, 2, 2)), ((48, 120, 216), (2, 2, 2)),
                                           ((60, 108, 212), (1, 2, 4))])
def test_not_finite_in_the_fused_steps(extent, factor, value):
    """A whole inference, whose finest level's first step reads the coarser
    state and whose last one writes the readout, against the upsample, the steps
    and the readout one after another."""
    n_in, steps = 3, (3, 2)
    wl = scaled(VIDEO_2DT, extent, n_in=n_in, factors=(factor,), steps=steps)
    weights = upload_weights(make_weights(wl, 3))
    model = octnca.Model(ndim=3, n_in=n_in, dtype="f16")
    image = torch.rand(extent + (n_in,), generator=torch.Generator("cuda").manual_seed(2),
                       device="cuda").half()
    for z, y, x in ((0, 0, 0), (extent[0] // 2, 11, 37), (extent[0] - 1, extent[1] - 1, 60)):
        image[z, y, x, 1] = value
    state, seg = Inference(model, extent, [factor])(image, weights, steps, 0.5, 1234)

    coarse_extent = tuple(e // f for e, f in zip(extent, factor))
    coarse = torch.zeros(coarse_extent + (16,), dtype=torch.float16, device="cuda")
    level = coarse[..., :n_in].contiguous()
    octnca.octree_nca_build_pyramid(model, image, [factor], [level])
    coarse[..., :n_in] = level
    other = torch.empty_like(coarse)
    octnca.octree_nca_run_level(model, coarse, other, weights[1], 1, steps[1], 0.5, 1234)
    b0 = torch.empty(extent + (16,), dtype=torch.float16, device="cuda")
    octnca.octree_nca_upsample(model, coarse, factor, image, b0)
    b1 = torch.empty_like(b0)
    octnca.octree_nca_run_level(model, b0, b1, weights[0], 0, steps[0], 0.5, 1234)
    want_seg = torch.empty(extent, dtype=torch.uint8, device="cuda")
    octnca.octree_nca_readout(model, b1, want_seg)
    torch.cuda.synchronize()
    assert not torch.isfinite(b1).all()
    assert torch.equal(_kinds(state), _kinds(b1))
    ok = torch.isfinite(b1)
    assert torch.equal(state[ok], b1[ok])
    assert torch.equal(seg, want_seg)
