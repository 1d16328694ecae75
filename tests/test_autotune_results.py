"""The autotuner's default search holds no field that a result depends on (no GPU)."""
import sys
import types

from paper_2106_12802_amd import autotune


def test_default_search_leaves_the_node_format_alone(monkeypatch, tmp_path):
    """Quantized and FP32 nodes may differ in a hit at a grazed box: tried where a caller
    lists the field, never by default, however fast."""
    state = dict.fromkeys(autotune.T.TUNING_KEYS, 0)
    tried = set()

    def set_tuning(**kw):
        state.update(kw)
        tried.add(state["bvh_quantized"])

    monkeypatch.setattr(autotune.T, "get_tuning", lambda: dict(state))
    monkeypatch.setattr(autotune.T, "set_tuning", set_tuning)
    monkeypatch.setattr(autotune, "_device_key", lambda: "fake")
    fake_torch = types.SimpleNamespace(cuda=types.SimpleNamespace(synchronize=lambda: None))
    monkeypatch.setitem(sys.modules, "torch", fake_torch)
    clock = [0.0]
    monkeypatch.setattr(autotune.time, "perf_counter", lambda: clock[0])

    def workload():  # quantized nodes twice as fast
        clock[0] += 2.0 - state["bvh_quantized"]

    path = str(tmp_path / "cache.json")
    res = autotune.tune(workload, "w", cache_path=path, reps=1, candidates=[(1, 1, 0)])
    assert tried == {0} and res["bvh_quantized"] == 0
    res = autotune.tune(workload, "v", cache_path=path, reps=1, candidates=[(1, 1, 0)],
                        secondary=[("bvh_quantized", (0, 1))])
    assert tried == {0, 1} and res["bvh_quantized"] == 1
