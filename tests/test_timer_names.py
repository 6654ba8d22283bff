"""The kernel timers that the benchmark asks for are those that the header names."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_benchmark_timers_exist():
    with open(os.path.join(ROOT, "include", "ofks.h")) as f:
        doc = re.search(r"Totals for a kernel class: name is one of(.*?)\(the host's", f.read(), re.S).group(1)
    named = set(re.findall(r'"(\w+)"', doc))
    with open(os.path.join(ROOT, "bench.py")) as f:
        asked = set(re.findall(r'"(\w+)"', re.search(r"P_STUDY_TIMERS = \((.*?)\)", f.read(), re.S).group(1)))
    assert asked and asked <= named, asked - named
