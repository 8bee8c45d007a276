"""The brick step (k_brick), which small boxes take by default: ragged bricks,
extents below a brick and down to one node, walls on every axis (at rest,
wetting, moving), every storage form and level format, and a batch, against
the FP64 oracle at the standard tolerances."""
import numpy as np
import pytest

from paper_1904_03618_amd import lbcg as B
from paper_1904_03618_amd import workloads as W
from gpu_helpers import gpu_run, oracle_run
from test_gpu_parity import _gpu, assert_parity  # noqa: F401  (_gpu: the module fixture)

pytestmark = pytest.mark.gpu


def _moving(case, wu):
    return dict(case[0], wall_u=wu), case[1]


CASES = {
    "periodic_ragged": lambda: W.random_state_case(33, 31, 17, seed=61, force=(1e-5, 0, 0)),
    "periodic_1x1x1": lambda: W.random_state_case(1, 1, 1, seed=62),
    "periodic_2x3x2": lambda: W.random_state_case(2, 3, 2, seed=63),
    "periodic_16x4x4": lambda: W.random_state_case(16, 4, 4, seed=64),
    "z_wetting_buoyancy": lambda: W.random_state_case(17, 9, 12, seed=65, bc=(0, 0, 1), theta=(65.0, 140.0),
                                                      grav=(0, 0, -1e-4), rho_ref=2.0),
    "z_one_layer_moving": lambda: _moving(W.random_state_case(18, 5, 1, seed=66, bc=(0, 0, 1), theta=(70.0, 100.0)),
                                          ((0.0, 0.01, 0.0), (0.02, 0.0, 0.0))),
    "z_moving": lambda: _moving(W.random_state_case(19, 7, 11, seed=67, bc=(0, 0, 1)),
                                ((0.03, 0.01, 0.0), (-0.02, 0.0, 0.0))),
    "y_wetting": lambda: W.random_state_case(21, 11, 13, seed=68, bc=(0, 1, 0), theta=(65.0, 140.0)),
    "y_moving": lambda: _moving(W.random_state_case(21, 4, 6, seed=69, bc=(0, 1, 0)),
                                ((0.02, 0.0, 0.01), (-0.01, 0.0, 0.0))),
    "x_wetting": lambda: W.random_state_case(19, 6, 5, seed=70, bc=(1, 0, 0), theta=(65.0, 140.0)),
    "x_one_layer": lambda: W.random_state_case(1, 6, 5, seed=71, bc=(1, 0, 0), theta=(80.0, 110.0)),
    "x_moving": lambda: _moving(W.random_state_case(18, 9, 6, seed=72, bc=(1, 0, 0)),
                                ((0.0, 0.02, 0.01), (0.0, -0.01, 0.0))),
}
STEPS = 200
_ORACLE = {}


def _oracle(name, p, fl):
    if name not in _ORACLE:
        _ORACLE[name] = oracle_run(p, fl, STEPS)
    return _ORACLE[name]


def _is_brick(case, **kw):
    h = B.lbcg_init([case], **kw)
    try:
        return B.lbcg_step_kernel(h) == "twopass" or B.lbcg_zchunk(h) == 4
    finally:
        B.lbcg_free(h)


@pytest.mark.parametrize("level", ["pair", "compact"])
@pytest.mark.parametrize("name", list(CASES))
def test_brick_step_matches_oracle(name, level):
    p, fl = CASES[name]()
    if level == "compact" and (p["bc"][0] or p["bc"][1]):
        level = "auto"                                 # pair levels, the walls' only format
    assert _is_brick((p, fl), level=level)
    g = gpu_run([(p, fl)], STEPS, level=level)[0]
    assert_parity(f"brick_{level}_{name}", g, _oracle(name, p, fl), p)


# the bounds of the 16-bit pair forms over 500 steps
@pytest.mark.parametrize("storage,tn,tu", [("fp16s", 6e-3, 2e-4), ("bf16s", 1e-1, 2e-3)])
@pytest.mark.parametrize("name", ["periodic_ragged", "z_wetting_buoyancy", "y_moving"])
def test_brick_step_in_16bit_forms(name, storage, tn, tu):
    p, fl = CASES[name]()
    g = gpu_run([(p, fl)], STEPS, storage=storage)[0]
    o = _oracle(name, p, fl)
    assert np.abs(g["rhoN"] - o["rhoN"]).max() <= tn
    assert max(np.abs(g[k] - o[k]).max() for k in ("ux", "uy", "uz")) <= tu


def test_brick_batch_of_mixed_walls_matches_oracle():
    names = ["periodic_ragged", "y_wetting", "z_wetting_buoyancy", "x_one_layer"]
    cases = [CASES[n]() for n in names]
    for name, g, (p, fl) in zip(names, gpu_run(cases, STEPS), cases):
        assert_parity(f"brick_batch_{name}", g, _oracle(name, p, fl), p)


def test_chunks_below_eight_planes_fill_the_workgroup_slots():
    """A 64^3 box has more than two bricks per CU and marches; 16 columns of
    tiles leave the 512 slots of the FP32 kernel idle at 8 planes, so the
    rule goes down to 2 (512 tiles), and the run matches explicit chunks to
    FP32 rounding (1e-6 relative after 20 steps: the same arithmetic per node)."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    case = W.random_state_case(64, 64, 64, seed=73, bc=(0, 0, 1))
    assert 4 * 16 * 16 > 2 * cus
    h = B.lbcg_init([case])
    try:
        best = min(range(1, 129), key=lambda zc: (-(-16 * -(-64 // zc) // (2 * cus)) * (zc + 2), -zc))
        assert B.lbcg_zchunk(h) == best
    finally:
        B.lbcg_free(h)
    a, b = gpu_run([case], 20)[0], gpu_run([case], 20, zchunk=16)[0]
    for k in ("rhoR", "rhoB", "ux", "uy", "uz"):
        scale = 3.0 if k.startswith("rho") else 0.1
        assert np.abs(a[k] - b[k]).max() <= 1e-6 * scale, k
