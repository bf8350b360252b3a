"""How the library's host code divides steps over launches (no GPU): the plans
are printed by a small host program linked against the built library."""
import os
import subprocess

import pytest

from paper_2508_06993_amd.build import CSRC, INCLUDE, LIB_NAME, PKG, hipcc

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def plans(library_path, tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plans") / "plan_probe")
    subprocess.run([hipcc(), "-std=c++17", "-O1", "-x", "hip", "--offload-host-only", "-I", INCLUDE,
                    "-I", CSRC, os.path.join(HERE, "plan_probe.cpp"), "-o", exe, "-L", PKG,
                    "-l:" + LIB_NAME, "-Wl,-rpath," + PKG], check=True)

    def ask(queries):
        text = "\n".join(" ".join(str(v) for v in q) for q in queries)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        rows = [tuple(int(v) for v in line.split()) for line in out.splitlines()]
        assert len(rows) == len(queries)
        return rows
    return ask


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("c,h", [(16, 64), (12, 48)])
def test_plans_of_a_given_parity(plans, dtype, c, h):
    """A run whose result has to be in one of two buffers takes the best plan
    among those with the parity of its steps: two launches of one step each are
    not used where one launch of one step is not."""
    sizes = [(1, 1), (64, 64), (128, 128), (320, 320), (512, 512), (600, 600), (700, 851),
             (774, 775), (40, 6000), (6000, 40), (333, 1001)]
    ask = lambda steps, parity: plans([("block", dtype, c, h, *s, steps, 1, parity) for s in sizes])
    one = ask(1, 0)
    for steps in (1, 2, 3, 4, 5, 8, 19, 20, 23):
        for free, same, single in zip(ask(steps, 0), ask(steps, 1), one):
            if same[0]:
                assert free[0]
                assert same[2] % 2 == steps % 2 and same[2] >= free[2] - 1
            if free[0] and free[2] % 2 == steps % 2:
                assert same == free
            if steps == 2:
                assert same[0] == single[0]


@pytest.mark.parametrize("rows,cols,steps,large", [
    (33, 61, 1, 0), (100, 128, 1, 0), (160, 160, 1, 0), (200, 220, 1, 1), (320, 320, 1, 1),
    (33, 61, 2, 1), (20, 20, 20, 1), (1, 1, 3, 1)])
def test_2d_backward_on_large_tiles(plans, rows, cols, steps, large):
    """One step of a small level runs on 64-cell blocks, where it is faster."""
    assert plans([("bwd", 2, 1, rows, cols, steps)])[0][0] == large


@pytest.mark.parametrize("d,rows,cols,large", [
    (12, 48, 48, 0), (8, 64, 64, 0), (16, 48, 48, 1), (24, 48, 48, 1), (4, 128, 128, 1),
    (5, 96, 96, 0), (6, 112, 112, 1), (12, 96, 96, 1), (2, 200, 200, 0), (1, 256, 256, 0),
    (2, 400, 400, 0), (7, 131, 129, 1), (24, 160, 160, 1)])
def test_3d_backward_on_large_tiles(plans, d, rows, cols, large):
    """The tiles are 4 planes deep: thin volumes leave them mostly empty and run
    on 64-cell blocks, as do volumes that leave most CUs idle."""
    for steps in (1, 4):
        assert plans([("bwd", 3, d, rows, cols, steps)])[0][0] == large


@pytest.mark.parametrize("d,rows,cols", [(12, 96, 96), (24, 160, 160), (24, 320, 320),
                                         (40, 400, 400), (101, 203, 307)])
def test_3d_backward_sums_few_tiles_in_fp32(plans, d, rows, cols):
    """A row of weight-gradient sums, kept in fp32, covers at most 8 tiles of 256
    cells however large the volume is; the rows are added in fp64."""
    tiles = -(-d // 4) * -(-rows // 8) * -(-cols // 8)
    use, _, _, sums = plans([("bwd", 3, d, rows, cols, 1)])[0]
    assert use and tiles <= 8 * sums and sums <= tiles


@pytest.mark.parametrize("dtype,c,h,d,rows,cols,special", [
    ("f16", 12, 48, 2, 200, 200, 0), ("f16", 12, 48, 2, 160, 160, 1), ("f16", 12, 48, 1, 500, 500, 1),
    ("f16", 12, 48, 3, 200, 200, 1), ("f32", 12, 48, 2, 200, 200, 1), ("f16", 16, 64, 2, 200, 200, 1),
    ("f16", 20, 100, 3, 200, 200, 0)])
def test_volumes_of_two_planes(plans, dtype, c, h, d, rows, cols, special):
    assert plans([("serves", dtype, c, h, d, rows, cols)])[0][0] == special


@pytest.mark.parametrize("d,rows,cols,run", [
    (14, 243, 64, 4), (57, 106, 32, 4), (34, 65, 40, 3), (22, 66, 56, 2), (4, 30, 304, 1),
    (1, 1, 1, 1), (60, 108, 212, 12), (48, 120, 216, 12), (1800, 240, 432, 106), (1800, 60, 108, 113)])
def test_runs_of_the_fp16_3d_step(plans, d, rows, cols, run):
    """Where it costs little, every work item has a CU of its own; the runs of
    large levels fill the block slots."""
    assert plans([("run", d, rows, cols)])[0][0] == run
