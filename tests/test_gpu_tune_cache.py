"""The batch planner's cache keeps what was measured on the kernels at hand: a
line stored for other kernels, or by a library that did not name them, is not
used."""
import json
import re

import pytest
import torch

from paper_2303_00301_amd import workloads as W
from tests.test_gpu_batch import _chains

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    from paper_2303_00301_amd import sampler
    return sampler


def test_cache_lines_belong_to_their_kernels(S, tmp_path):
    ws = W.ragged_poisson_batch(n_chains=3, n_min=40, n_max=90, dims=(8,), seed=31)
    chains = _chains(S, ws, 1)
    cache = tmp_path / "tune.jsonl"

    def planned():  # the block of a new plan, and whether the cache had it
        before = cache.read_text() if cache.exists() else ""
        plan = S.BatchPlan(chains, 1, block=0, tune_cache=str(cache))
        (cls,) = plan.info()["classes"]
        plan.close()
        return cls["block"], cache.read_text() == before

    block, cached = planned()
    (line,) = cache.read_text().splitlines()
    assert not cached and json.loads(line)["block"] == block
    assert re.fullmatch("[0-9a-f]{16}", json.loads(line)["kernels"])
    other = 3  # no candidate of the search
    line = re.sub(r'"block": \d+', f'"block": {other}', line)
    cache.write_text(line + "\n")
    assert planned() == (other, True)
    for foreign in (re.sub(r'"kernels": "\w+"', '"kernels": "0123456789abcdef"', line),
                    re.sub(r'"kernels": "\w+", ', "", line)):
        assert foreign != line
        cache.write_text(foreign + "\n")
        got, cached = planned()
        assert got != other and not cached
    torch.cuda.synchronize()
