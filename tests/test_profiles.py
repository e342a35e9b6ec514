"""Committed profiles and the bench lines built on them are of kernels that exist: what replaces a kernel has its
counters taken again, or the bench would print another kernel's traffic."""
import glob
import json
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _kernels():
    names = set()
    for f in glob.glob(os.path.join(ROOT, "paper_2309_03523_amd", "csrc", "*.hip")):
        names |= set(re.findall(r"\b__global__\b[^;{]*?\b(k_\w+)\s*\(", open(f).read()))
    return names


def test_profiles_name_present_kernels():
    kernels = _kernels()
    assert {"k_dense_split", "k_rows_split", "k_agg", "k_dw_split", "k_gat_dx"} <= kernels
    table = json.load(open(os.path.join(ROOT, "profiles", "hbm_traffic.json")))
    sources = [e["source"] for e in table.values() if isinstance(e, dict) and "source" in e] + ["profiles/timed_cases_kernel_times.txt"]
    assert len(sources) > 6
    for src in sources:
        named = set(re.findall(r"(?<!\w)(k_[a-z]\w*)", open(os.path.join(ROOT, src)).read()))
        assert named and not named - kernels, (src, sorted(named - kernels))
    notes = " ".join(v for k, v in table.items() if isinstance(v, str)) + " ".join(e.get("_note", "") for e in table.values() if isinstance(e, dict))
    assert not set(re.findall(r"(?<!\w)(k_[a-z]\w*)", notes)) - kernels


def test_bench_names_present_kernels():
    named = set(re.findall(r"(?<!\w)(k_[a-z]\w*)", open(os.path.join(ROOT, "bench.py")).read()))
    assert named and not named - _kernels(), sorted(named - _kernels())
