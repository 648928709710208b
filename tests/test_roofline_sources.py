"""Stored traffic counters are reported only for the sources they were taken on, headers included."""
import json

import pytest

from paper_1908_11848_amd import roofline


@pytest.mark.parametrize("srcs,changed", [("_CONV_SRCS", "common.hpp"), ("_CONV_SRCS", "bn_merge.hpp"), ("_CONV_SRCS", "k_conv.hip"), ("_BN_SRCS", "common.hpp"),
                                          ("_SERVER_SRCS", "common.hpp"), ("_SERVER_SRCS", None)])
def test_counters_of_other_sources(monkeypatch, tmp_path, srcs, changed):
    srcs = getattr(roofline, srcs)
    db = {"source_hash": {s: roofline.source_hash(s) for s in srcs}, "kernels": {"a": {"fetch_bytes": 2, "write_bytes": 1}}}
    if changed:
        db["source_hash"][changed] = "another"
    (tmp_path / "c.json").write_text(json.dumps(db))
    monkeypatch.setattr(roofline, "_COUNTERS", str(tmp_path / "c.json"))
    assert roofline._traffic("a", srcs) == (None if changed else 3)
    assert set(srcs) <= set(roofline.SOURCES)
