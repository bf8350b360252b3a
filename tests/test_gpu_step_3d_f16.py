"""The fp16 3D step's perception on the matrix cores (step_3d_f16.hip): one
step and several against the vector kernel, whose perception sums the same
fp16 states and fp32 taps one by one in fp32, at sizes around its 8 x 32 tiles,
2 x 8 blocks and plane runs; and cells that are not finite, which must reach
their own 3 x 3 x 3 neighbours only.

Bound: one step rounds taps, perception, features and hidden units to fp16
(2^-11 each) and stores fp16; sums of 27 and 32 products of N(0, 1) states keep
the relative error of the largest value below 8 * 2^-11 = 4e-3 (five steps:
sqrt(5) times that, below 1e-2)."""
import pytest
import torch

import paper_2508_06993_amd as octnca
from paper_2508_06993_amd.runtime import upload_weights
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
                                   (7, 17, 66), (300, 3, 5), (37, 24, 100), (4, 10, 34)])
@pytest.mark.parametrize("steps", [1, 5])
def test_steps_match_vector_kernel(shape, n_in, steps):
    weights, state = _setup(shape, n_in)
    got = _run("mfma", state, weights, n_in, steps).float()
    want = _run("valu", state, weights, n_in, steps).float()
    assert torch.isfinite(got).all()
    tol = 4e-3 if steps == 1 else 1e-2
    assert float((got - want).abs().max()) <= tol * max(1.0, float(want.abs().max()))
    assert torch.equal(got[..., :n_in], state.float()[..., :n_in])


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
def test_values_that_are_not_finite_stay_local(value):
    shape, n_in = (6, 21, 70), 3
    weights, state = _setup(shape, n_in)
    clean = _run("mfma", state, weights, n_in, 1, rate=1.0).float()
    spots = [(0, 0, 0), (3, 10, 33), (5, 20, 69), (2, 4, 8)]
    near = torch.zeros(shape, dtype=torch.bool, device="cuda")
    dirty = state.clone()
    for z, y, x in spots:
        dirty[z, y, x, 7] = value
        near[max(0, z - 1):z + 2, max(0, y - 1):y + 2, max(0, x - 1):x + 2] = True
    got = _run("mfma", dirty, weights, n_in, 1, rate=1.0).float()
    assert torch.isfinite(got[~near]).all()
    assert float((got - clean)[~near].abs().max()) <= 4e-3 * float(clean.abs().max())
    # the same cells are touched as by the vector kernel
    for z, y, x in spots:
        assert not torch.isfinite(got[z, y, x]).all()
