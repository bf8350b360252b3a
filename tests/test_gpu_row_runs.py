"""How the 2D row kernel divides a level into runs of rows: one run a SIMD, two
or three (fp16, rows off 8-cell boundaries), as many as runs of 128 rows take.
The tile kernel sums in the same order and knows no runs, so every division has
to give its bits; sizes lie on both sides of each rule's line."""
import pytest
import torch

import paper_2508_06993_amd as octnca
from paper_2508_06993_amd.runtime import upload_weights
from synthetic import TINY_2D, make_weights, scaled

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("shape", [(1020, 512), (1025, 513), (1217, 512), (1219, 515),
                                   (961, 1341), (8193, 520), (8199, 517)])
def test_runs_give_the_tile_kernels_bits(shape, dtype):
    wl = scaled(TINY_2D, (1,) + shape, dtype=dtype, factors=(), steps=(1,))
    weights = upload_weights(make_weights(wl, 3))[0]
    gen = torch.Generator(device="cuda").manual_seed(7)
    out = []
    for kernel in ("mfma_rows,mfma_1step", "mfma_tiles"):
        model = octnca.Model(ndim=2, n_in=wl.n_in, dtype=dtype, kernel=kernel)
        gen.manual_seed(7)
        b0 = torch.randn((1,) + shape + (16,), generator=gen, device="cuda").to(model.torch_dtype)
        b1 = torch.full_like(b0, float("nan"))
        assert octnca.octree_nca_run_level(model, b0, b1, weights, 1, 3, 0.5, 99) == 1
        torch.cuda.synchronize()
        out.append(b1)
    assert torch.equal(out[0].view(torch.uint8), out[1].view(torch.uint8))
