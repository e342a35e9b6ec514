"""bench.py's command line and its one JSON line: run in this process (no child process), on the
smallest workload."""
import importlib.util
import json
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _bench():
    spec = importlib.util.spec_from_file_location("bench_under_test", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def test_more_than_one_gpu_is_refused_with_a_message(monkeypatch, capsys):
    monkeypatch.setattr(sys, "argv", ["bench.py", "--gpus", "2"])
    with pytest.raises(SystemExit) as ei:
        _bench().main()
    assert ei.value.code not in (0, None)
    assert "one GPU" in capsys.readouterr().err


@pytest.mark.gpu
def test_json_line_of_the_smallest_workload(monkeypatch, capsys):
    monkeypatch.setattr(sys, "argv", ["bench.py", "--workload", "config1", "--steps", "5", "--warmup", "2",
                                      "--cpu-seconds", "1"])
    _bench().main()
    lines = [ln for ln in capsys.readouterr().out.splitlines() if ln.strip()]
    assert len(lines) == 1                       # exactly one line on stdout
    d = json.loads(lines[0])
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
                "vs_baseline", "dtype", "data", "config", "roofline", "cpu_baseline"):
        assert key in d, key
    assert d["n_gpus"] == 1 and d["steps"] == 5 and d["warmup"] == 2
    assert d["higher_is_better"] is True and d["vs_baseline"] is None and d["data"] == "synthetic"
    assert d["dtype"] == "f32" and "workload" in d["config"] and "model" not in d["config"]
    assert d["value"] > 0 and d["ms_per_step"] > 0
    r = d["roofline"]
    for key in ("bound", "achieved", "peak", "unit", "frac", "traffic"):
        assert key in r, key
    assert r["bound"] in ("hbm", "mfma", "alu") and r["peak"] > 0
    assert abs(r["frac"] - r["achieved"] / r["peak"]) < 1e-9 * max(1.0, r["frac"])
    c = d["cpu_baseline"]
    for key in ("value", "unit", "cores", "kind", "sample"):
        assert key in c, key
    assert c["kind"] == "oracle" and c["value"] > 0 and c["cores"] >= 1
    assert c["gpu_max_rel_err_on_sample"] < 1e-4


def test_dense_kernel_rules_are_the_librarys():
    """What the roofline names and counts is what the library's own rules choose, over widths, tiles and windows on either side."""
    import ctypes as ct
    lib = ct.CDLL(os.path.join(ROOT, "paper_2309_03523_amd", "libdgc.so"))
    fold, narrow = lib._ZN3dgc17dense_fold_wantedEiii, lib._ZN3dgc19dense_narrow_wantedEiibli
    fold.restype = narrow.restype = ct.c_bool
    fold.argtypes, narrow.argtypes = [ct.c_int32] * 3, [ct.c_int32, ct.c_int32, ct.c_bool, ct.c_int64, ct.c_int32]
    b = _bench()
    for kind, code in (("gru", 1), ("lstm", 2)):
        for S in range(32, 257, 32):
            for K0 in range(1, 305):
                folds = b.folds_transform(K0, S, kind)
                assert folds == fold(S, K0, code), (kind, S, K0)
                if S > 64:
                    assert not b.runs_narrow(K0, S, kind, 1, 8)
                    continue
                for tiles in (1, 64, 65, 128, 129, 192, 256, 257, 384, 512, 513, 640, 641, 768, 769, 1024, 1025, 2047, 2048, 100000):
                    for window in (1, 2, 3, 4, 5, 32):
                        assert b.runs_narrow(K0, S, kind, tiles, window) == narrow(S, K0, folds, tiles, window), (kind, S, K0, tiles, window)
