"""The line that bench.py prints on stdout: the contract's fields whole, the
measured ones unrounded, and short enough to be kept; the other legs stay out."""
import json

import bench


def test_headline_holds_the_contract_and_is_short():
    value, ms = 18012345678.123457, 0.36412345678901234
    per = {n: {k: 1.0 / 3 * i for i, k in enumerate(("ms_mean", "ms_p50", "ms_p99", "kernel_ms_mean", "tri_per_s",
                                                      "invocations", "shading_rate", "reuse", "speedup_vs_naive",
                                                      "hbm_frac", "alu_frac"))} for n in ("plan", *bench.KERNEL_NAMES)}
    line = {k: k for k in bench.HEADLINE}
    line.update(value=value, ms_per_step=ms, n_gpus=1, steps=20, warmup=5, vs_baseline=None, per_strategy=per,
                config={"workload": "w", "strategies": list(bench.KERNEL_NAMES)}, roofline={"frac": 2.0 / 3, "traffic": None},
                sweep=[{"ms": 1.0 / 7}] * 1000, scene={"draws": list(range(5000))})
    text = bench.headline(line)
    out = json.loads(text)
    assert "\n" not in text and len(text) < 3000
    assert out["value"] == value and out["ms_per_step"] == ms
    assert set(out) == set(bench.HEADLINE)
    for key in ("metric", "unit", "n_gpus", "steps", "warmup", "higher_is_better", "scaling", "vs_baseline", "dtype",
                "data", "config"):
        assert out[key] == line[key]
    assert out["roofline"]["frac"] == 0.666667 and out["per_strategy"]["naive"]["ms_p50"] == 0.333333


def test_significant_keeps_what_is_no_finite_float():
    x = {"a": [float("inf"), 1, True, None, "1.23456789"], "b": (0.0, -1.23456789e-7)}
    assert bench.significant(x) == {"a": [float("inf"), 1, True, None, "1.23456789"], "b": [0.0, -1.23457e-7]}
