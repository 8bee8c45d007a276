"""The marching step (k_fused) with several tiles per workgroup, whose LDS rings are
reused from tile to tile, down to chunks of one plane, and the brick step in the
16-bit forms; against the FP64 oracle at the standard tolerances.  (Small boxes run
bricks unless a chunk is given, so the chunk is given here.)"""
import numpy as np
import pytest

from paper_1904_03618_amd import lbcg as B
from paper_1904_03618_amd import workloads as W
from gpu_helpers import gpu_run, oracle_run
from test_gpu_parity import _gpu, assert_parity  # noqa: F401  (_gpu: the module fixture)

pytestmark = pytest.mark.gpu

STEPS = 100


def _moving(case):
    return dict(case[0], wall_u=((0.02, 0.01, 0.0), (-0.015, 0.02, 0.0))), case[1]


CASES = {
    "periodic": lambda: W.random_state_case(40, 19, 11, seed=91, force=(1e-5, 0, 0)),
    "z_wetting": lambda: W.random_state_case(37, 17, 9, seed=92, bc=(0, 0, 1), theta=(65.0, 140.0)),
    "z_moving": lambda: _moving(W.random_state_case(35, 18, 10, seed=93, bc=(0, 0, 1), theta=(70.0, 110.0))),
    "z_one_layer_moving": lambda: _moving(W.random_state_case(34, 9, 1, seed=94, bc=(0, 0, 1), theta=(70.0, 100.0))),
}
_ORACLE = {}


def _oracle(name, p, fl):
    if name not in _ORACLE:
        _ORACLE[name] = oracle_run(p, fl, STEPS)
    return _ORACLE[name]


# the bounds of the 16-bit pair forms over 500 steps
BOUNDS = {"fp16s": (6e-3, 2e-4), "bf16s": (1e-1, 2e-3)}


def _close(g, o, storage):
    tn, tu = BOUNDS[storage]
    assert np.abs(g["rhoN"] - o["rhoN"]).max() <= tn
    assert max(np.abs(g[k] - o[k]).max() for k in ("ux", "uy", "uz")) <= tu


@pytest.mark.parametrize("level", ["pair", "compact"])
@pytest.mark.parametrize("zchunk", [1, 4])
@pytest.mark.parametrize("name", list(CASES))
def test_marching_tiles_in_few_workgroups(name, zchunk, level):
    p, fl = CASES[name]()
    opt = dict(kernel="fused", zchunk=zchunk, level=level)
    tiles = -(-p["nx"] // 32) * -(-p["ny"] // 8) * -(-p["nz"] // zchunk)
    g = gpu_run([(p, fl)], STEPS, **opt)[0]
    assert_parity(f"march_{level}_{zchunk}_{name}", g, _oracle(name, p, fl), p)
    for blocks in (1, 3):
        assert blocks < tiles
        few = gpu_run([(p, fl)], STEPS, persistent_blocks=blocks, **opt)[0]
        for k in ("rhoR", "rhoB", "ux", "uy", "uz"):
            assert np.array_equal(few[k], g[k]), (blocks, k)


@pytest.mark.parametrize("storage", list(BOUNDS))
def test_marching_batch_in_few_workgroups_16bit(storage):
    cases = [CASES[n]() for n in CASES]
    got = gpu_run(cases, STEPS, storage=storage, kernel="fused", zchunk=1, persistent_blocks=5)
    for name, g, (p, fl) in zip(CASES, got, cases):
        _close(g, _oracle(name, p, fl), storage)


@pytest.mark.parametrize("storage", list(BOUNDS))
@pytest.mark.parametrize("name", list(CASES))
def test_bricks_in_16_bits(name, storage):
    p, fl = CASES[name]()
    h = B.lbcg_init([(p, fl)], storage=storage)
    try:
        assert (B.lbcg_step_kernel(h), B.lbcg_zchunk(h)) == ("fused", 4)
    finally:
        B.lbcg_free(h)
    g = gpu_run([(p, fl)], STEPS, storage=storage)[0]
    _close(g, _oracle(name, p, fl), storage)
    few = gpu_run([(p, fl)], STEPS, storage=storage, persistent_blocks=2)[0]
    for k in ("rhoR", "rhoB", "ux", "uy", "uz"):
        assert np.array_equal(few[k], g[k]), k
