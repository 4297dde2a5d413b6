"""bench.py's kernel figures describe the launches that were timed."""
import json

import pytest

import bench

ARGS = dict(ndof=1 << 20, M=4, dim=2, N=3, stages=4, flux=1, precision="fp64", ms_step=0.06)


def _times(plain, blend, local):
    return {"k_local_plain_ms": plain, "k_local_blend_ms": blend, "empty_interval_ms": 0.005, "interface_ms": 0.025,
            "local_phase_ms": local}


@pytest.fixture
def profile(tmp_path, monkeypatch):
    """A profile summary of one workload taken with the current sources."""
    rec = {"workload": "w", "kernel": "crk::k_local_any<double, 2, 3, 1, 4, 1, 4>", "kernel_instance": "plain",
           "sources_sha256": bench.sources_digest(), "hbm_bytes": 1.0e8, "fp64_flops": 1.0e9}
    (tmp_path / "profiles").mkdir()
    (tmp_path / "profiles" / "p.md").write_text("counters: " + json.dumps(rec) + "\n")
    digest = rec["sources_sha256"]
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    monkeypatch.setattr(bench, "sources_digest", lambda: digest)
    return rec


def test_one_launch_for_every_tile(profile):
    r = bench.kernel_report("w", _times(0.042, None, 0.0425), **ARGS)
    assert r["kernel"] == "local stages, the launch of every tile: " + profile["kernel"]
    assert r["kernel_ms"] == 0.042 and r["local_phase_ms"] == 0.0425 and r["other_launch_ms"] is None
    assert r["traffic"] == profile["hbm_bytes"]


def test_two_launches(profile):
    r = bench.kernel_report("w", _times(0.042, 0.012, 0.050), **ARGS)
    assert r["kernel"].startswith("local stages, the launch of the tiles that cannot blend")
    assert r["kernel_ms"] == 0.042 and r["other_launch_ms"] == 0.012 and r["local_phase_ms"] == 0.050
    # counters of the other kind's kernel are not attached
    r = bench.kernel_report("w", _times(0.012, 0.042, 0.050), **ARGS)
    assert r["kernel"] == "local stages, the launch of the tiles that can blend" and r["traffic"] is None


def test_no_profile_no_name():
    r = bench.kernel_report("no such workload", _times(0.042, None, 0.0425), **ARGS)
    assert r["kernel"] == "local stages, the launch of every tile" and r["counter_profile"] is None


def test_digest_covers_the_local_stages_kernels():
    """the files that hold k_local, k_local_any and k_local_split"""
    assert {f.rsplit("/", 1)[1] for f in bench.KERNEL_SOURCES} >= {"crk_kernels.hpp", "crk_physics.hpp", "crk_split.hpp"}
