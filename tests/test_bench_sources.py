"""bench.py reports measured traffic only if it was taken on the sources that decide it: the pair passes and
the list builds, with every local header that they include."""
import os
import re

import bench

CSRC = os.path.join(bench.ROOT, "paper_2107_07315_amd", "csrc")


def test_digest_covers_the_passes_and_the_list_builds():
    named = {os.path.basename(f) for f in bench.KERNEL_SOURCES}
    kernels = ("k_density(", "k_forces(", "k_build_tiles(", "k_tile_split(", "k_tile_flags(")
    want = {f for f in os.listdir(CSRC) if f.endswith(".hip")
            and any("void " + k in open(os.path.join(CSRC, f)).read() or "\n" + k in open(os.path.join(CSRC, f)).read()
                    for k in kernels)}
    assert {"sph_pairs.hip", "sph_cells.hip", "sph_cellgrid.hip"} <= want <= named
    for f in sorted(want):
        for h in re.findall(r'#include "(sph_(?:build|listout|internal)\.h)"', open(os.path.join(CSRC, f)).read()):
            assert h in named, (f, h)


def test_traffic_of_other_sources_is_not_reported(monkeypatch):
    monkeypatch.setattr(bench, "sources_digest", lambda: "0" * 16)
    assert bench.measured_traffic("k_forces<float>") is None
