"""The generic step kernel's fifth channel quad (C = 20, H = 100: step_gen.hip)
against the vector kernel, at sizes around its 8 x 32 and 2 x 4 x 32 tiles, with
more tiles than the blocks that run them have fire bits formed ahead for; and
states that are not finite, which must stay within their own neighbourhoods
(unused product slots hold zeros, and zero times infinity would be NaN).

Bound: fp32 states run on fp16 operands with split weights: features and
hidden units keep 11 bits of their layer's range; 40 and 100 of them sum to an
error below 4e-3 of the largest value for one step (fp16 states store 11 bits
on top).  Five steps: sqrt(5) times that, below 1e-2."""
import pytest
import torch

import paper_2508_06993_amd as octnca
from paper_2508_06993_amd.runtime import upload_weights
import numpy as np
from synthetic import TINY_2D, VIDEO_2DT, LevelWeights, make_weights, scaled

pytestmark = pytest.mark.gpu

C, H = 20, 100


def _setup(shape, dtype, seed=4):
    rng = np.random.default_rng(seed)
    taps = 9 if shape[0] == 1 else 27
    w = LevelWeights(
        conv_w=rng.normal(0, taps ** -0.5, (C, taps)).astype(np.float32),
        conv_b=rng.normal(0, 0.1, (C,)).astype(np.float32),
        w1=rng.normal(0, (2 * C) ** -0.5, (H, 2 * C)).astype(np.float32),
        b1=rng.normal(0, 0.1, (H,)).astype(np.float32),
        w2=rng.normal(0, 0.5 * H ** -0.5, (C, H)).astype(np.float32))
    gen = torch.Generator(device="cuda").manual_seed(seed)
    state = torch.randn(shape + (C,), generator=gen, device="cuda")
    return upload_weights([w])[0], state.half() if dtype == "f16" else state


def _run(kernel, state, weights, n_in, steps, rate=0.5):
    model = octnca.Model(ndim=2 if state.shape[0] == 1 else 3, n_in=n_in, channels=C, hidden=H,
                         dtype="f16" if state.dtype == torch.float16 else "f32", kernel=kernel)
    b0, b1 = state.clone(), torch.full_like(state, float("nan"))
    at = octnca.octree_nca_run_level(model, b0, b1, weights, 1, steps, rate, 77)
    torch.cuda.synchronize()
    return b1 if at else b0


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("n_in", [1, 3])
@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 8, 32), (1, 9, 33), (1, 7, 31), (1, 40, 65),
                                   (1, 1203, 997), (2, 4, 32), (3, 5, 33), (2, 3, 31),
                                   (9, 70, 100), (24, 61, 130)])
def test_steps_match_vector_kernel(shape, n_in, dtype):
    weights, state = _setup(shape, dtype)
    for steps, tol in ((1, 4e-3), (5, 1e-2)):
        got = _run("mfma", state, weights, n_in, steps).float()
        want = _run("valu", state, weights, n_in, steps).float()
        assert torch.isfinite(got).all()
        assert float((got - want).abs().max()) <= tol * max(1.0, float(want.abs().max()))
        assert torch.equal(got[..., :n_in], state.float()[..., :n_in])


@pytest.mark.parametrize("n_in", [1, 3])
@pytest.mark.parametrize("shape", [(2, 160, 160), (2, 181, 179), (2, 200, 200), (3, 181, 179)])
def test_two_planes_of_the_small_model(shape, n_in):
    """fp16 12/48 volumes on both sides of the line from which two planes run on
    the generic kernel."""
    wl = scaled(VIDEO_2DT, shape, n_in=n_in, channels=12, hidden=48, factors=(), steps=(1,))
    weights = upload_weights(make_weights(wl, 3))[0]
    gen = torch.Generator(device="cuda").manual_seed(3)
    state = torch.randn(shape + (12,), generator=gen, device="cuda").half()
    out = {}
    for kernel in ("mfma", "valu"):
        model = octnca.Model(ndim=3, n_in=n_in, channels=12, hidden=48, dtype="f16", kernel=kernel)
        b0, b1 = state.clone(), torch.full_like(state, float("nan"))
        assert octnca.octree_nca_run_level(model, b0, b1, weights, 1, 5, 0.5, 77) == 1
        torch.cuda.synchronize()
        out[kernel] = b1.float()
    got, want = out["mfma"], out["valu"]
    assert torch.isfinite(got).all()
    assert float((got - want).abs().max()) <= 1e-2 * max(1.0, float(want.abs().max()))
    assert torch.equal(got[..., :n_in], state.float()[..., :n_in])


def test_rows_too_wide_for_the_specialised_step():
    """fp32 12/48 volumes whose 18 rows of 64-byte cells pass 2^32 bytes run on
    the generic kernel, whose offsets are within 2 x 4 x 32 tiles."""
    shape = (1, 1, 3_800_003)
    assert 18 * 64 * shape[2] >= 2 ** 32
    wl = scaled(VIDEO_2DT, shape, n_in=1, channels=12, hidden=48, dtype="f32", factors=(),
                steps=(1,))
    weights = upload_weights(make_weights(wl, 3))[0]
    gen = torch.Generator(device="cuda").manual_seed(3)
    state = torch.randn(shape + (12,), generator=gen, device="cuda")
    out = []
    for kernel in ("mfma", "valu"):
        model = octnca.Model(ndim=3, n_in=1, channels=12, hidden=48, kernel=kernel)
        b0, b1 = state.clone(), torch.full_like(state, float("nan"))
        assert octnca.octree_nca_run_level(model, b0, b1, weights, 1, 1, 0.5, 77) == 1
        torch.cuda.synchronize()
        out.append(b1)
    got, want = out
    assert torch.isfinite(got).all()
    assert float((got - want).abs().max()) <= 4e-3 * max(1.0, float(want.abs().max()))
    assert torch.equal(got[..., :1], state[..., :1])


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("channel", [2, 17])   # a full quad's, the last quad's
def test_values_that_are_not_finite_stay_local(value, channel):
    weights, state = _setup((1, 21, 70), "f32")
    clean = _run("mfma", state, weights, 1, 1, rate=1.0)
    dirty = state.clone()
    near = torch.zeros((1, 21, 70), dtype=torch.bool, device="cuda")
    for y, x in ((0, 0), (10, 33), (20, 69), (4, 8)):
        dirty[0, y, x, channel] = value
        near[0, max(0, y - 1):y + 2, max(0, x - 1):x + 2] = True
    got = _run("mfma", dirty, weights, 1, 1, rate=1.0)
    assert torch.equal(got[~near], clean[~near])


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("shape", [(1, 33, 61), (1, 333, 451), (1, 1025, 800)])
def test_layouts_of_the_small_model_give_the_same_bits(shape, dtype):
    """The 12/48 model's 2D steps: tiles kept on chip or rows as the size asks,
    rows, and the generic kernel's tiles sum in the same order and round once."""
    wl = scaled(TINY_2D, shape, n_in=3, channels=12, hidden=48, dtype=dtype, factors=(), steps=(1,))
    weights = upload_weights(make_weights(wl, 3))[0]
    out = []
    for kernel in ("mfma", "mfma_rows,mfma_1step", "mfma_tiles"):
        model = octnca.Model(ndim=2, n_in=3, channels=12, hidden=48, dtype=dtype, kernel=kernel)
        gen = torch.Generator(device="cuda").manual_seed(7)
        b0 = torch.randn(shape + (12,), generator=gen, device="cuda").to(model.torch_dtype)
        b1 = torch.full_like(b0, float("nan"))
        assert octnca.octree_nca_run_level(model, b0, b1, weights, 1, 3, 0.5, 99) == 1
        torch.cuda.synchronize()
        out.append(b1)
    for other in out[1:]:
        assert torch.equal(out[0].view(torch.uint8), other.view(torch.uint8))
