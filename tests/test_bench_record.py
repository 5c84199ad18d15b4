"""The benchmark's record of measured traffic is tied to every source that the
single-qdot kernels are built from."""
import os

import bench


def test_sources_of_every_single_qdot_route_are_hashed():
    names = {os.path.basename(p) for p in bench.kernel_sources()}
    assert {"qdot_kernels.hip", "qdot_fused.hip", "qdot_device.hpp", "qdot_blocks.hpp",
            "qdot_select.hpp", "qdot_guess.hpp"} <= names
    assert all(os.path.isfile(p) for p in bench.kernel_sources())


def test_a_change_in_any_of_them_is_seen(monkeypatch, tmp_path):
    before = bench.kernel_source_sha()
    for p in bench.kernel_sources():
        copy = tmp_path / os.path.basename(p)
        copy.write_bytes(open(p, "rb").read() + b"\n// changed\n")
        paths = [str(copy) if s == p else s for s in bench.kernel_sources()]
        with monkeypatch.context() as m:
            m.setattr(bench, "kernel_sources", lambda: paths)
            assert bench.kernel_source_sha() != before
