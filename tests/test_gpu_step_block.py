"""Several steps of a small 2D level in one launch (step_block.hip).

The launches run the same operations in the same order as one launch per step
(kernel "mfma_1step"), so every result must be the same bits: on grids smaller
than a tile, on ragged edges, rows that start inside an 8-cell fire block, odd
and even step counts (the result's buffer), fire rates 0 and 1, and whole
inferences, whose first launch of a level also forms the upsampled state or
the seed and whose last one writes the readout.
"""
import pytest
import torch

import paper_2508_06993_amd as octnca
from paper_2508_06993_amd.runtime import Inference, upload_weights
from synthetic import TINY_2D, make_image, make_weights, scaled

pytestmark = pytest.mark.gpu

KINDS = [("f32", 16, 64), ("f32", 12, 48), ("f16", 16, 64), ("f16", 12, 48)]


def _models(dtype, c, h, n_in):
    k = dict(ndim=2, n_in=n_in, dtype=dtype, channels=c, hidden=h)
    return octnca.Model(**k), octnca.Model(kernel="mfma_1step", **k)


def _bits(t):
    return t.contiguous().view(torch.uint8)


def _level(model, state, weights, steps, rate):
    b0, b1 = state.clone(), torch.full_like(state, float("nan"))
    at = octnca.octree_nca_run_level(model, b0, b1, weights, 2, steps, rate, 12345)
    torch.cuda.synchronize()
    assert at == steps % 2
    return b1 if at else b0


@pytest.mark.parametrize("dtype,c,h", KINDS)
@pytest.mark.parametrize("shape", [(1, 1), (3, 70), (16, 16), (33, 61), (64, 40), (130, 131),
                                   (257, 250), (9, 2000), (700, 851)])
def test_levels_equal_single_steps(dtype, c, h, shape):
    n_in = 1 if shape[0] % 2 else 3
    wl = scaled(TINY_2D, (1,) + shape, channels=c, hidden=h, n_in=n_in, dtype=dtype, factors=(),
                steps=(1,))
    weights = upload_weights(make_weights(wl, 3))[0]
    block, single = _models(dtype, c, h, n_in)
    gen = torch.Generator(device="cuda").manual_seed(7)
    state = torch.randn((1,) + shape + (c,), generator=gen, device="cuda").to(block.torch_dtype)
    for steps, rate in ((1, 0.5), (2, 1.0), (7, 0.5), (20, 0.5), (23, 0.4), (4, 0.0)):
        want = _level(single, state, weights, steps, rate)
        got = _level(block, state, weights, steps, rate)
        assert torch.equal(_bits(got), _bits(want)), (steps, rate)


@pytest.mark.parametrize("dtype,c,h", KINDS)
@pytest.mark.parametrize("extent,factors,steps", [
    ((1, 64, 64), ((1, 2, 2), (1, 2, 2)), (10, 10, 10)),
    ((1, 90, 126), ((1, 3, 2), (1, 5, 7)), (3, 11, 6)),       # uneven factors, ragged levels
    ((1, 48, 400), ((1, 8, 8), (1, 1, 5)), (5, 0, 9)),        # a level without steps between
    ((1, 700, 640), ((1, 2, 2), (1, 2, 2)), (4, 5, 6)),       # the finest level past the limit
    ((1, 7, 5), (), (12,)),
])
def test_inference_equals_single_steps(dtype, c, h, extent, factors, steps):
    wl = scaled(TINY_2D, extent, steps=steps, channels=c, hidden=h, factors=factors, dtype=dtype)
    weights = upload_weights(make_weights(wl, 5))
    image = torch.from_numpy(make_image(wl, 5)).cuda()
    out = []
    for model in _models(dtype, c, h, 3):
        run = Inference(model, extent, factors)
        run.state.fill_(float("nan"))
        run.seg.fill_(7)
        state, seg = run(image, weights, steps, 0.5, 99)
        torch.cuda.synchronize()
        out.append((state.clone(), seg.clone()))
    assert torch.equal(_bits(out[0][0]), _bits(out[1][0]))
    assert torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("extent", [(1, 40, 72), (1, 104, 100)])
def test_training_forward_equals_single_steps(extent):
    """The training forward writes every state between the steps; its last one
    is that of an inference with the same operands, one step per launch."""
    factors, steps = ((1, 2, 2), (1, 2, 2)), (7, 5, 6)
    wl = scaled(TINY_2D, extent, steps=steps, factors=factors)
    weights = upload_weights(make_weights(wl, 8))
    image = torch.from_numpy(make_image(wl, 8)).cuda()
    run = Inference(octnca.Model(ndim=2, n_in=3, kernel="mfma_bf16x3"), extent, factors)
    want, _ = run(image, weights, steps, 0.5, 4)
    model = octnca.Model(ndim=2, n_in=3)
    n = octnca.octree_nca_train_workspace_bytes(model, extent, factors, steps)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    grads = [{k: torch.empty_like(v) for k, v in w.items()} for w in weights]
    got = torch.empty_like(want)
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    target = torch.zeros(extent + (2,), device="cuda")
    octnca.octree_nca_train_step(model, image, factors, weights, steps, 0.5, 4, target, ws, grads,
                                 loss, got)
    torch.cuda.synchronize()
    assert torch.equal(_bits(got), _bits(want))
