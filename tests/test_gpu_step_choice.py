"""Which step a handle runs, what it reports of it, and that walled boxes give the
same bits however they are launched: alone, in a batch, with other launch
options, and continued from a checkpoint in a handle with other options."""
import pytest

from paper_1904_03618_amd import lbcg as B
from paper_1904_03618_amd import workloads as W
from test_gpu_parity import _gpu  # noqa: F401  (the module fixture)

pytestmark = pytest.mark.gpu

STEPS = 12


def _moving(case, wu):
    return dict(case[0], wall_u=wu), case[1]


WALLED = {
    "y_rest": lambda: W.random_state_case(20, 12, 9, seed=81, bc=(0, 1, 0)),
    "y_wetting": lambda: W.random_state_case(21, 11, 13, seed=82, bc=(0, 1, 0), theta=(65.0, 140.0)),
    "y_moving": lambda: _moving(W.random_state_case(33, 9, 6, seed=83, bc=(0, 1, 0)),
                                ((0.02, 0.0, 0.01), (-0.01, 0.0, 0.0))),
    "x_wetting": lambda: W.random_state_case(19, 6, 5, seed=84, bc=(1, 0, 0), theta=(65.0, 140.0)),
    "x_one_layer": lambda: W.random_state_case(1, 6, 5, seed=85, bc=(1, 0, 0), theta=(80.0, 110.0)),
    "x_moving": lambda: _moving(W.random_state_case(18, 9, 6, seed=86, bc=(1, 0, 0)),
                                ((0.0, 0.02, 0.01), (0.0, -0.01, 0.0))),
}
OTHERS = {
    "periodic": lambda: W.random_state_case(20, 12, 9, seed=87),
    "z_moving": lambda: _moving(W.random_state_case(20, 12, 9, seed=88, bc=(0, 0, 1)),
                                ((0.02, 0.01, 0.0), (0.0, -0.01, 0.0))),
}


def _run(cases, steps=STEPS, load=None, save=False, **opt):
    """Populations of every case (and the checkpoint image), the step kernel, the
    chunk and the kernels that the timing recorded."""
    h = B.lbcg_init(cases, **opt)
    try:
        if load is not None:
            B.lbcg_checkpoint_load(h, load)
        B.lbcg_timing(h, not opt.get("graph_steps"))
        B.lbcg_step(h, steps)
        ran = {k for k, (_, n) in B.lbcg_timing_read(h).items() if n}
        f = [B.lbcg_get_populations(h, c).cpu() for c in range(len(cases))]
        return f, B.lbcg_step_kernel(h), B.lbcg_zchunk(h), ran, B.lbcg_checkpoint_save(h) if save else None
    finally:
        B.lbcg_free(h)


@pytest.mark.parametrize("storage", ["fp32", "fp16s", "bf16s"])
@pytest.mark.parametrize("name", list(WALLED))
def test_walls_on_x_or_y_run_the_two_pass_step(name, storage):
    import torch
    case = WALLED[name]()
    f, kernel, zc, ran, _ = _run([case], storage=storage)
    assert (kernel, zc, ran) == ("twopass", 0, {"aux", "ghost", "collide"})
    big = W.random_state_case(140, 140, 20, seed=89, bc=(0, 1, 0))
    moving = case[0] if any(v for s in case[0]["wall_u"] for v in s) else None
    for cases, opt in (([case], dict(kernel="twopass")), ([case], dict(block_nodes=128)),
                       ([case], dict(block_nodes=64, persistent_blocks=3)), ([case], dict(graph_steps=4)),
                       ([case], dict(zchunk=4)), ([case, case], {})):
        for g in _run(cases, storage=storage, **opt)[0]:
            assert torch.equal(g, f[0]), opt
    if moving is None:                       # (a batch with a moving case runs that case's instance)
        assert torch.equal(_run([case, big], storage=storage)[0][0], f[0])


@pytest.mark.parametrize("name", list(WALLED))
def test_walled_checkpoints_continue_bit_for_bit_under_other_options(name):
    import torch
    case = WALLED[name]()
    whole = _run([case], 2 * STEPS)[0][0]
    image = _run([case], STEPS, save=True)[4]
    for opt in ({}, dict(block_nodes=128), dict(persistent_blocks=2), dict(zchunk=4), dict(kernel="twopass")):
        assert torch.equal(_run([case], STEPS, load=image, **opt)[0][0], whole), opt


@pytest.mark.parametrize("name", list(OTHERS))
def test_small_boxes_of_the_fused_step_run_bricks(name):
    """Reported as the fused step with chunks of 4 planes (16-bit compact levels
    march); an explicit chunk marches."""
    case = OTHERS[name]()
    for opt in (dict(), dict(level="pair"), dict(storage="fp16s"), dict(storage="bf16s"), dict(persistent_blocks=3)):
        assert _run([case], **opt)[1:4] == ("fused", 4, {"fused"}), opt
    assert _run([case], zchunk=3)[1:4] == ("fused", 3, {"fused"})
    assert _run([case], kernel="twopass")[1:3] == ("twopass", 0)


@pytest.mark.parametrize("storage", ["fp16s", "bf16s"])
def test_moving_walls_in_16_bits_march_two_workgroups_per_cu(storage):
    """The moving-wall instance of 16-bit pairs holds two workgroups per CU in
    its registers (three made it spill): the default chunk is the rule's for two."""
    import torch
    slots = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    case = _moving(W.random_state_case(128, 64, 128, seed=90, bc=(0, 0, 1)), ((0.02, 0.01, 0.0), (0.0, -0.01, 0.0)))
    tiles = lambda zc: 4 * 8 * -(-128 // zc)
    assert tiles(64) < 2 * slots
    best = min(range(1, 65), key=lambda zc: (-(-tiles(zc) // slots) * (zc + 2), -zc))
    h = B.lbcg_init([case], storage=storage)
    try:
        assert (B.lbcg_step_kernel(h), B.lbcg_zchunk(h)) == ("fused", best)
    finally:
        B.lbcg_free(h)
