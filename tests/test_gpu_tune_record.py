"""Tuning records hold for the kernels that were timed: one without their tag, or with another, is timed again."""
import json
import re

import pytest

from gpu_helpers import problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
E = pytest.importorskip("paper_2511_01793_amd.emagpie")


@pytest.mark.parametrize("other", ["", "kernels=0123456789abcdef "])
def test_record_of_other_kernels_is_not_used(tmp_path, other):
    print("case: tune record", repr(other), flush=True)
    p = problem("tiny", n=2 * 64 + 9, m=64, scan=("raster", 3, 34, 1), photons=1e6, B=1, L=1, alpha=0.05, seed=29)
    cache = str(tmp_path / "tune.jsonl")

    def tuned():
        d = torch.from_numpy(p.intensities).cuda()
        rec = E.Reconstruction(p.positions, d, p.n, minibatch=1, path="auto", tune_cache=cache)
        plan = rec.plan
        rec.close()
        return plan["tuned"]

    assert tuned() == "timed" and tuned() == "cache"
    record = json.loads(open(cache).read())
    key = re.sub(r"kernels=\w+ ", other, record["key"])
    open(cache, "w").write(json.dumps({**record, "key": key}) + "\n")
    assert tuned() == "timed" and tuned() == "cache"
