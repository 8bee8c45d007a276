"""The launch-shape autotuner may not return something slower than no tuning: the
fused step's own default is among what it times, and a choice cached before the
kernels changed is not reused (host logic, no GPU)."""
import json

from paper_1904_03618_amd import autotune as AT
from paper_1904_03618_amd import lbcg as B
from paper_1904_03618_amd import workloads as W


def _timed(monkeypatch, cases, ms, **kw):
    """autotune with the timing replaced by ms(options); the options it timed and
    the number of cases it timed them on."""
    seen = []

    def time_config(_, sample, storage, opts, **_kw):
        seen.append((len(sample), opts))
        return ms(opts)
    monkeypatch.setattr(AT, "time_config", time_config)
    monkeypatch.setattr(B, "load", lambda: None)
    return AT.autotune(cases, cache=None, **kw), seen


def test_the_default_of_the_fused_step_is_timed_and_can_win(monkeypatch):
    cases = [W.random_state_case(6, 5, 4, seed=1)]
    default = lambda o: o["kernel"] == "fused" and o["zchunk"] == 0
    (best, _), seen = _timed(monkeypatch, cases, lambda o: 1.0 if default(o) else 2.0)
    assert default(best)
    assert sorted(o["graph_steps"] for _, o in seen if default(o)) == [0, 8]


def test_the_default_is_left_out_where_a_sample_stands_for_the_batch(monkeypatch):
    """Bricks or the slot-filling chunk of 8 boxes say nothing of 64."""
    cases = [W.random_state_case(6, 5, 4, seed=1)] * 64
    (best, _), seen = _timed(monkeypatch, cases, lambda o: 1.0 + o["graph_steps"])
    assert {n for n, _ in seen} == {8}
    assert all(o.get("zchunk", 1) for _, o in seen)


def test_walls_on_x_or_y_leave_the_fused_step_out(monkeypatch):
    _, seen = _timed(monkeypatch, [W.random_state_case(6, 5, 4, seed=1, bc=(0, 1, 0))], lambda o: 1.0)
    assert seen and all(o["kernel"] == "twopass" for _, o in seen)


def test_cached_choices_of_other_kernels_are_not_reused(monkeypatch, tmp_path):
    cases = [W.random_state_case(6, 5, 4, seed=1)]
    cache = tmp_path / "cache.json"
    old = {"kernel": "fused", "zchunk": 64, "persistent_blocks": 0, "graph_steps": 0}
    # the key as it was without a version
    key = "fp32|cases=1|walls=0|side=4-6|nodes=120"
    assert AT.box_class(cases, "fp32").endswith(key) and AT.box_class(cases, "fp32") != key
    cache.write_text(json.dumps({key: {"options": old}}))
    monkeypatch.setattr(AT, "time_config", lambda *a, **kw: 1.0)
    best, rep = AT.autotune(cases, "fp32", cache=str(cache))
    assert not rep["cached"] and best != old
    assert AT.autotune(cases, "fp32", cache=str(cache))[1]["cached"]
