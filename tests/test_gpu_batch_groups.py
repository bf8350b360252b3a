"""Batches whose images share launches (coarse levels of a group of images
together, the finest level in parts): every image of the batch must be what
the batch gives with one step per launch, image after image (kernel
"mfma_1step"), bit for bit.  Batch sizes that leave parts of one image, a
single level, uneven factors, a finest level past the shared launches' limit,
step counts of both parities (the last image's coarse state sits in its own
final state) and a workspace larger than needed; large images whose levels are
worth sharing for many steps and not for one.  The 20/100 model has no
multi-step launches and runs image by image: its images against the vector
kernel's (their fire masks follow the image's index; fp32 states on fp16
operands, 40 and 100 products of 11 bits a step, up to 30 steps: below 1e-2 of
the largest value) and the first against a single inference.
"""
import pytest
import torch

import paper_2508_06993_amd as octnca
from paper_2508_06993_amd.runtime import Inference, upload_weights
from synthetic import TINY_2D, make_weights, scaled

pytestmark = pytest.mark.gpu


def _batch(model, images, factors, weights, steps, extra=0):
    ext = tuple(images.shape[1:4])
    n = octnca.octree_nca_workspace_bytes(model, ext, factors, True) + extra
    ws = torch.full((n,), 255, dtype=torch.uint8, device="cuda")
    states = torch.full(images.shape[:4] + (model.channels,), float("nan"), device="cuda",
                        dtype=model.torch_dtype)
    segs = torch.full(images.shape[:4], 9, dtype=torch.uint8, device="cuda")
    octnca.octree_nca_infer_batch(model, images, factors, weights, steps, 0.5, 31, ws, states,
                                  segs)
    torch.cuda.synchronize()
    return states, segs


@pytest.mark.parametrize("dtype,c,h", [("f32", 16, 64), ("f16", 16, 64), ("f32", 12, 48),
                                       ("f32", 20, 100)])
@pytest.mark.parametrize("batch,hw,factors,steps", [
    (2, (64, 64), ((1, 2, 2), (1, 2, 2)), (10, 10, 10)),
    (3, (40, 56), ((1, 2, 2),), (1, 6)),                       # one launch on the finest level
    (8, (48, 80), ((1, 2, 2), (1, 2, 2), (1, 2, 2)), (5, 7, 3, 11)),
    (5, (17, 23), (), (9,)),                                   # no coarse level
    (7, (30, 42), ((1, 1, 1), (1, 3, 7)), (4, 3, 8)),          # level 1 as large as level 0
    (4, (36, 60), ((1, 2, 2), (1, 3, 5)), (6, 0, 5)),          # a level without steps
    (3, (700, 640), ((1, 2, 2), (1, 2, 2)), (3, 4, 5)),        # the finest level image by image
    (70, (8, 16), ((1, 2, 2),), (3, 12)),                      # more than one group
    (2, (2048, 1536), ((1, 2, 2),) * 3, (1, 1, 1, 1)),         # too few steps to share
    (3, (1024, 768), ((1, 2, 2),) * 3, (2, 9, 10, 8)),
])
def test_batch_equals_single_steps(dtype, c, h, batch, hw, factors, steps):
    wl = scaled(TINY_2D, (1,) + hw, steps=steps, channels=c, hidden=h, factors=factors,
                dtype=dtype)
    weights = upload_weights(make_weights(wl, 6))
    k = dict(ndim=2, n_in=3, dtype=dtype, channels=c, hidden=h)
    group = octnca.Model(**k)
    single = octnca.Model(kernel="mfma_1step" if c != 20 else "valu", **k)
    gen = torch.Generator(device="cuda").manual_seed(batch)
    images = torch.rand((batch, 1) + hw + (3,), generator=gen, device="cuda").to(group.torch_dtype)
    want = _batch(single, images, factors, weights, steps)
    for extra in (0, 1 << 20):
        got = _batch(group, images, factors, weights, steps, extra)
        if c == 20:
            scale = want[0].abs().amax(dim=(1, 2, 3, 4))
            assert bool(((got[0] - want[0]).abs().amax(dim=(1, 2, 3, 4)) <= 1e-2 * scale).all())
            first, seg = Inference(group, (1,) + hw, factors)(images[0], weights, steps, 0.5, 31)
            assert torch.equal(got[0][0], first) and torch.equal(got[1][0], seg)
            continue
        assert torch.equal(got[0].view(torch.uint8), want[0].view(torch.uint8))
        assert torch.equal(got[1], want[1])
