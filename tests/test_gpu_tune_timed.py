"""Launch shapes: a batch large enough for the tuner to time its candidates stores
what it chose, and shapes of a tuning file -- more waves per workgroup, longer
items, half of the CUs -- give the same results, with shared waves and apart."""
import json
import os
import subprocess
import sys

import pytest

from gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_CHILD = r"""
import json, sys
import numpy as np
import torch
sys.path.insert(0, sys.argv[1])
from paper_2108_02419_amd import _bbe, inputs
B, sims = 17_000, int(sys.argv[2])
rng = np.random.default_rng(1)
race = _bbe.Race(inputs.competitor_params(rng, 3), inputs.TRACK_LEN)
wins = torch.zeros((B, 20), dtype=torch.int64, device="cuda")
tab = _bbe.RequestTable([race] * B, sims, np.arange(B), 1)
plan = _bbe.BatchPlan(tab, 5, wins, autotune=True)
got, infos = [], [plan.info()]
where = np.arange(B) * 5 // B
for states in (None, where):
    if states is not None:
        pos = (100.0 + 10.0 * states[:, None] + np.arange(3)).astype(np.float32)
        plan.set_states(20 + states.astype(np.uint32), pos, np.full((B, 3), 6.0, np.float32))
        infos.append(plan.info())
    plan.launch()
    torch.cuda.synchronize()
    got.append(int((wins * torch.arange(1, 20 * B + 1, device="cuda").view(B, 20)).sum().item()))
print(json.dumps(dict(infos=infos, got=got)))
"""


@pytest.mark.parametrize("sims", [64, 3])
def test_timed_and_given_shapes(tmp_path, sims):
    require_gpu()
    cache = tmp_path / "tune.json"

    def child(what):
        announce(f"launch shapes, {sims} simulations a request: {what}")
        out = subprocess.run([sys.executable, "-c", _CHILD, ROOT, str(sims)], timeout=180,
                             env=dict(os.environ, BBE_TUNE_CACHE=str(cache)),
                             capture_output=True, text=True, check=True).stdout
        return json.loads(out.strip().splitlines()[-1])

    first = child("tuned")
    entry, = json.loads(cache.read_text())["entries"]
    assert entry["sims_per_item"] == first["infos"][0]["sims_per_item"]
    assert entry["sims_per_item"] in ((64, 128) if sims == 64 else (64,))
    for shape in ((4, 128, 1), (2, 192, 2)):
        given = dict(entry, waves_per_block=shape[0], sims_per_item=shape[1], cu_share=shape[2])
        cache.write_text('{"entries": [\n  ' + json.dumps(given) + "\n]}\n")
        second = child(f"given {shape}")
        for info in second["infos"]:
            assert (info["waves_per_block"], info["sims_per_item"]) == shape[:2]
        assert second["got"] == first["got"]
