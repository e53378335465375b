"""The tag of the kernels in the tuning records' key follows every source, header and flag."""
import os
import shutil

from paper_2511_01793_amd.csrc import build as b

HEADER = os.path.join(b.ROOT, "include", "emagpie.h")


def test_tag_follows_the_sources(tmp_path, monkeypatch):
    here = tmp_path / "csrc"
    shutil.copytree(b.HERE, here, ignore=shutil.ignore_patterns("_build", "__pycache__"))
    header = tmp_path / "emagpie.h"
    shutil.copy(HEADER, header)
    tag = b.source_tag(str(here), str(header))
    assert tag == b.source_tag() and len(tag) == 16
    seen = {tag}
    for path in [here / f for f in b.SOURCES + ["kernels.hpp", "kernels_chain.hpp", "plans.hpp"]] + [header]:
        kept = path.read_bytes()
        path.write_bytes(kept + b"\n")
        seen.add(b.source_tag(str(here), str(header)))
        path.write_bytes(kept)
    assert len(seen) == 1 + len(b.SOURCES) + 4
    assert b.source_tag(str(here), str(header)) == tag
    monkeypatch.setattr(b, "HIPFLAGS", b.HIPFLAGS + ["-O2"])
    assert b.source_tag() != tag
