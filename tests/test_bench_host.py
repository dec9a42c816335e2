"""Host-side pieces of bench.py: the kernel-source hash that ties the
recorded HBM counters (profiles/traffic.json) to the code they were taken
on follows the code and ignores its comments."""
from __future__ import annotations

import os
import shutil

import bench

SRC = ("ks_kernels.hip", "ks_expand.hip", "ks_internal.h", "ks_sched.inc")


def _tree(tmp_path, edit=None):
    d = tmp_path / "paper_2606_28565_amd" / "csrc"
    d.mkdir(parents=True)
    for f in SRC:
        shutil.copy(os.path.join(bench.ROOT, "paper_2606_28565_amd", "csrc", f), d / f)
    if edit:
        p = d / "ks_kernels.hip"
        p.write_text(edit(p.read_text()))
    return str(tmp_path)


def _hash(monkeypatch, root):
    monkeypatch.setattr(bench, "ROOT", root)
    return bench.kernel_source_hash()


def test_source_hash_ignores_comments_and_blank_lines(tmp_path, monkeypatch):
    base = _hash(monkeypatch, _tree(tmp_path / "a"))
    commented = _hash(monkeypatch, _tree(tmp_path / "b", lambda s: "// note\n\n/* block\n comment */\n" +
                                         s.replace("\n}\n", "\n}  // end\n\n", 3)))
    assert commented == base


def test_source_hash_follows_code(tmp_path, monkeypatch):
    base = _hash(monkeypatch, _tree(tmp_path / "a"))
    changed = _hash(monkeypatch, _tree(tmp_path / "b", lambda s: s.replace("kStreamR * lane", "kStreamR*lane", 1)))
    assert changed != base


def test_fp32_peak_is_six_products_of_pieces():
    """An fp32 head product is six bfloat16 ones: 704,000 pairs of the 32-128 head in
    167 us (174 TFLOP/s) are a share of the peak, not more than it."""
    assert bench.PEAK["f32"] == bench.PEAK["bf16"] / 6
    assert 0.3 < 704e3 * bench.head_flops_per_pair(32, 128) / 167e-6 / bench.PEAK["f32"] < 1


def test_evaluated_records_by_family():
    """The different records of the families that the call takes, every record of
    the others; on the MLP those outside the bounded families."""
    import torch
    # GEMM: 2 different of 6; grouped: 4; decode: 3 of 6 (by step); RMSNorm: 1 of 5 (no K)
    fam = [0] * 6 + [2] * 4 + [4] * 6 + [5] * 5
    fam_off = [sum(x < f for x in fam) for f in range(11)]
    t = {"m": [1, 2] * 3 + [0] * 4 + [0] * 6 + [7] * 5, "n": [64] * 21,
         "k": [8] * 16 + [1, 2, 3, 4, 5], "a": [0] * 10 + [2] * 6 + [0] * 5,
         "step": [0, 0, 1, 1, 2, 2] + [0, 1, 2, 2] + [0, 0, 1, 1, 2, 2] + [0, 0, 1, 1, 2]}
    t = {k: torch.tensor(v, dtype=torch.int32) for k, v in t.items()}
    every = (1 << 0) | (1 << 4) | (1 << 5)
    assert bench.evaluated_records(t, fam_off, every) == (2 + 4 + 3 + 1, 2 + 4 + 3 + 1)
    assert bench.evaluated_records(t, fam_off, 0) == (21, 21)
    assert bench.evaluated_records(t, fam_off, every, bounded=1 << 4) == (10, 7)
    assert bench.evaluated_records(t, fam_off, 1 << 0, bounded=1 << 0) == (17, 15)
