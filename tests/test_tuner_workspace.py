"""The tuner writes the FP16 values alone: the header's rows of the other precisions size
workspaces and come back as they are, with the header's own text."""
import os
import re

import pytest

from paper_1810_11359_amd import autotune

HEADER = os.path.join(os.path.dirname(autotune.__file__), "csrc", "ism_tuning.h")


def test_committed_header_is_the_writers(tmp_path):
    """The committed header is what write_header makes of the FP16 results that it states."""
    text = open(HEADER).read()
    res, waves = {}, {}
    for m in re.finditer(r"// W=(\d+) fp16 nS<=(\d+) \((.*?)\): best (\S+) / (\S+), score (\S+), "
                         r"default 1.2e5 / 49152 score (\S+)", text):
        best = (float(m[4]), float(m[5]))
        score = {(1.2e5, 49152.0): float(m[7])}
        score[best] = float(m[6])
        res[(int(m[1]), "fp16", int(m[2]))] = (best, score, {}, m[3].split(", "))
    for m in re.finditer(r"// W=(\d+) fp16 batch: best (\d+) waves per SIMD, items <= (\d+) taps; (.*)", text):
        grid = {(int(k), float(it)): float(v) for k, it, v in re.findall(r"\((\d+), (\d+)\): ([\d.]+)", m[4])}
        waves[(int(m[1]), "fp16")] = ((int(m[2]), float(m[3])), grid)
    assert len(res) == 12 and len(waves) == 1
    p = tmp_path / "ism_tuning.h"
    autotune.write_header(res, waves, str(p), re.search(r"target GPU \((.*)\)", text)[1])
    assert p.read_text() == text


def test_workspace_rows_are_not_tuned():
    with pytest.raises(ValueError):
        autotune.tune(precisions=("fp32",))
    rows = re.findall(r"\{(\d+), 0, (\d+), ([\d.e+]+), ([\d.]+)\}", open(HEADER).read())
    assert {(int(w), int(n)): (float(a), float(b)) for w, n, a, b in rows} == autotune.WORKSPACE_ROWS
