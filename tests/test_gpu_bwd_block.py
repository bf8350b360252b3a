"""The backward on large tiles (bwd_block.hip): one step against the oracle at
sizes that the larger tiles divide badly (ragged 2D tiles, more tiles than
CUs, a 3D level past the size from which its tiles are used), and a level's
steps, several per launch with a shrinking halo, against the same steps one
call at a time.

Bounds as in test_gpu_train.py: fp32 sums of a few dozen products per cell for
state gradients (2e-5 of the largest), fp32 sums over a block's cells for
weight gradients (1e-4).  The steps of a level compared call by call differ
only in the order of fp32 sums; a state gradient carried through t steps adds
t such errors (20 steps: 20 * 2e-5 / sqrt(20), below 1e-4)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2508_06993_amd as octnca
from paper_2508_06993_amd.runtime import upload_weights
from parity import max_rel_err, to_np
from test_gpu_train import (C, KEYS, TOL_STATE, TOL_WEIGHT, rand_weights, step_backward_gpu,
                            zero_grads)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ndim,n_in,shape", [
    (2, 3, (1, 45, 70)), (2, 1, (1, 333, 325)), (2, 3, (1, 2, 300)), (2, 3, (1, 70, 3)),
    (3, 1, (11, 75, 77)), (3, 3, (4, 137, 121))])
def test_step_matches_oracle(gpu, ndim, n_in, shape):
    rng = np.random.default_rng(17)
    w = rand_weights(rng, ndim)
    s = rng.normal(0, 1, shape + (C,)).astype(np.float32)
    g_out = rng.normal(0, 1, shape + (C,)).astype(np.float32)
    model = octnca.Model(ndim=ndim, n_in=n_in)
    gin, grads, _ = step_backward_gpu(model, s, g_out, w, 1, 3, 0.5, 21)
    want_in, want = oracle.step_vjp(s, w, n_in, ndim, 1, 3, 21, 0.5, g_out)
    assert max_rel_err(gin, want_in) <= TOL_STATE
    for k in KEYS:
        assert max_rel_err(grads[k], getattr(want, k) if not isinstance(want, dict) else want[k]) \
            <= TOL_WEIGHT, k


@pytest.mark.parametrize("n_in,shape", [(3, (1, 179, 181)), (1, (1, 2, 16100)), (3, (1, 11000, 3))])
def test_2d_step_past_the_one_step_line(gpu, n_in, shape):
    """Single steps take the large tiles from 32000 cells on: thin and ragged
    ones of that size."""
    test_step_matches_oracle(gpu, 2, n_in, shape)


@pytest.mark.parametrize("n_in,shape", [(1, (11, 60, 61)), (3, (4, 143, 133)), (1, (12, 80, 77))])
def test_3d_step_on_large_tiles(gpu, n_in, shape):
    """Ragged volumes that fill the 4 x 8 x 8 tiles well enough to take them:
    fewer tiles than CUs, more."""
    test_step_matches_oracle(gpu, 3, n_in, shape)


def test_3d_level_on_large_tiles(gpu):
    test_level_equals_its_steps(gpu, 3, 1, (11, 90, 84), 3, 0.5)


def test_3d_sums_over_many_tiles(gpu):
    """Weight gradients of a volume of 40000 tiles whose terms have one sign (no
    cancellation: a long fp32 sum shows its error): every cell fires, every
    hidden unit is active, so the sums are linear in G' and their fp64 values
    follow from those of G' and G' S^T.  The result's own rounding to fp32 is up
    to 2^-24 of it.  What the sums add: a row's 2048 cells, 4 a product and 8
    waves apart, are some 64 roundings of up to 2^-25 each, sqrt(64) * 2^-25 =
    2^-22 a row, and the 5000 rows are added in fp64: 2^-22 / sqrt(5000) = 2^-28."""
    shape = (64, 400, 400)
    rng = np.random.default_rng(5)
    w = rand_weights(rng, 3)
    for k in KEYS:
        setattr(w, k, np.abs(getattr(w, k)) * 0.1)
    state = torch.rand(shape + (C,), device="cuda", generator=torch.Generator("cuda").manual_seed(4))
    g_out = torch.rand(shape + (C,), device="cuda", generator=torch.Generator("cuda").manual_seed(5))
    model = octnca.Model(ndim=3, n_in=1)
    ws = torch.empty(octnca.octree_nca_step_backward_workspace_bytes(model, shape),
                     dtype=torch.uint8, device="cuda")
    grads, gin = zero_grads(w), torch.empty_like(g_out)
    octnca.octree_nca_step_backward(model, state, g_out, upload_weights([w])[0], 0, 0, 1.0, 1, gin,
                                    grads, ws)
    # per cell gu = G' (hidden channels), ga = W2^T gu, gP = (W1^T ga)_perception
    w1, w2 = (torch.from_numpy(v).cuda().double() for v in (w.w1, w.w2))
    gu = g_out.double()
    gu[..., :1] = 0
    gu_sum = gu.reshape(-1, C).sum(0)
    ga_sum = w2.T @ gu_sum
    want = {"b1": ga_sum, "conv_b": (w1.T @ ga_sum)[C:]}
    # dW1's state columns: sum of ga S^T
    f = state.double().reshape(-1, C)
    want_w1 = w2.T @ (gu.reshape(-1, C).T @ f)
    torch.cuda.synchronize()
    for k, v in want.items():
        assert max_rel_err(to_np(grads[k]), to_np(v)) <= 2.0 ** -24 + 2.0 ** -28, k
    assert max_rel_err(to_np(grads["w1"])[:, :C], to_np(want_w1)) <= 2.0 ** -24 + 2.0 ** -28


@pytest.mark.parametrize("ndim,n_in,shape,steps,rate", [
    (2, 3, (1, 20, 20), 20, 0.5), (2, 1, (1, 61, 45), 7, 1.0), (2, 3, (1, 170, 150), 5, 0.5),
    (2, 3, (1, 321, 318), 3, 0.4), (2, 3, (1, 9, 32), 4, 0.5), (2, 3, (1, 1, 40), 3, 0.5),
    (3, 1, (9, 90, 84), 3, 0.5), (3, 3, (5, 20, 21), 3, 0.5)])
def test_level_equals_its_steps(gpu, ndim, n_in, shape, steps, rate):
    rng = np.random.default_rng(23)
    host = rand_weights(rng, ndim, scale=0.1)
    w = upload_weights([host])[0]
    model = octnca.Model(ndim=ndim, n_in=n_in)
    exact = octnca.Model(ndim=ndim, n_in=n_in, kernel="mfma_bf16x3")
    image = torch.rand(shape + (n_in,), device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    target = torch.rand(shape + (2,), device="cuda", generator=torch.Generator("cuda").manual_seed(2))
    got = zero_grads(host)
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    ws = torch.empty(octnca.octree_nca_train_workspace_bytes(model, shape, [], [steps]),
                     dtype=torch.uint8, device="cuda")
    final = torch.empty(shape + (C,), device="cuda")
    octnca.octree_nca_train_step(model, image, [], [w], [steps], rate, 77, target, ws, [got], loss,
                                 final)

    seed_state = torch.zeros(shape + (C,), device="cuda")
    seed_state[..., :n_in] = image

    def state_before(t):
        b0, b1 = seed_state.clone(), torch.empty_like(seed_state)
        return b1 if octnca.octree_nca_run_level(exact, b0, b1, w, 0, t, rate, 77) else b0
    last = state_before(steps)
    assert torch.equal(last, final)
    g = torch.zeros_like(last)
    g[..., -2:] = last[..., -2:] - target
    want = zero_grads(host)
    bws = torch.empty(octnca.octree_nca_step_backward_workspace_bytes(model, shape),
                      dtype=torch.uint8, device="cuda")
    for t in range(steps - 1, -1, -1):
        octnca.octree_nca_step_backward(model, state_before(t), g, w, 0, t, rate, 77, g, want, bws)
    torch.cuda.synchronize()
    for k in KEYS:
        assert max_rel_err(to_np(got[k]), to_np(want[k])) <= 1e-4, k
