"""Host logic of bench.py: which committed traffic record a bench line may use."""
import json
import os
import shutil

import bench


def test_traffic_keys_separate_the_launch_shapes():
    base = bench.traffic_key("l32_32k", 1024, 64, False)
    keys = {base,
            bench.traffic_key("l32_32k", 1024, 64, True),
            bench.traffic_key("l32_32k", 1024, 32, False),
            bench.traffic_key("l32_32k", 1024, 64, False, shared_layers=3),
            bench.traffic_key("l32_32k", 1024, 64, False, schedule=1),
            bench.traffic_key("l32_32k", 1024, 64, False, schedule=2)}
    assert len(keys) == 6
    assert base == "l32_32k_b1024_w64"  # the default line's record keeps its key


def test_recorded_traffic_only_for_recorded_shapes():
    path = os.path.join(bench.ROOT, "profiles", "traffic.json")
    recorded = set(json.load(open(path)))
    # shared-index mode sweeps 3 layers: it must not pick up the 32-layer record
    assert bench.traffic_key("l32_32k", 1024, 64, False, shared_layers=3) not in recorded
    assert bench.recorded_traffic(bench.traffic_key("l32_32k", 1024, 64, False,
                                                    shared_layers=3)) is None
    for key in recorded:
        rec = json.load(open(path))[key]
        assert rec["hbm_bytes_per_launch"] == rec["fetch_bytes_per_launch"] + rec["write_bytes_per_launch"]


def test_traffic_records_follow_every_source_of_the_sweeps(tmp_path, monkeypatch):
    """An edit to the sweeps, their chunk lookup or the planning makes the records stale."""
    src = os.path.join(bench.ROOT, "paper_2609_22158_amd", "csrc")
    dst = tmp_path / "paper_2609_22158_amd" / "csrc"
    shutil.copytree(src, dst)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    start = bench.source_digest()
    for name in ("saliency.hip", "saliency_chunks.h", "api.cpp", "internal.h", "common.h"):
        text = (dst / name).read_bytes()
        (dst / name).write_bytes(text + b"\n// edited")
        assert bench.source_digest() != start, name
        (dst / name).write_bytes(text)
    assert bench.source_digest() == start


def test_saliency_form_counts_the_passes_over_k():
    assert bench.saliency_form(256, False, 0)[0] == 2
    assert bench.saliency_form(256, True, 0)[0] == 1
    # at most 8 window rows keep their logits, unless a schedule is forced
    assert bench.saliency_form(4, False, 0)[0] == bench.saliency_form(8, False, 0)[0] == 1
    assert bench.saliency_form(9, False, 0)[0] == 2
    assert bench.saliency_form(4, False, 1)[0] == bench.saliency_form(4, False, 2)[0] == 2
