"""The batched forward by its kernels: cached choices belong to the kernels they
were timed with (round trips and corrupt files: test_batched_gpu.py), and every
form handles waves outside the common batch inversion's range."""
import json
import re

import pytest

import oracle
from paper_2008_11326_amd import build
from paper_2008_11326_amd import inputs as I
from tests.gpu_helpers import assert_parity, mixed_pole_problem, say, to_device
from tests.test_batched_gpu import _tune_proc

pytestmark = pytest.mark.gpu


def test_a_choice_timed_with_other_kernels_is_not_taken(tmp_path):
    cache = tmp_path / "tune.json"
    first = _tune_proc(cache)
    assert first["tuned"] == 1 and first["from_cache"] == 0
    (key, entry), = json.loads(cache.read_text()).items()
    assert f":k={build.kernels_id()}:" in key
    for other in (re.sub(r":k=\w+", "", key), re.sub(r":k=\w+", ":k=00000000", key)):
        cache.write_text(json.dumps({other: entry}))
        again = _tune_proc(cache)
        assert again["from_cache"] == 0 and again["tuned"] == 1, other
        saved = json.loads(cache.read_text())
        assert set(saved) == {other, key}  # the other build's entry stays
    assert _tune_proc(cache)["from_cache"] == 1


@pytest.mark.parametrize("nw", range(1, 9))
@pytest.mark.parametrize("sched", [0, 2, 4])
def test_real_poles_in_every_batched_form(nw, sched, monkeypatch):
    """States with real and exact poles, vanishing om and many occupied bands in
    the persistent, queue and flat kernels."""
    import torch
    import paper_2008_11326_amd as gpp
    monkeypatch.setenv("GPP_BATCHED_SCHEDULE", str(sched))
    probs = [mixed_pole_problem(60 + k, d, f) for k, (d, f) in enumerate(
        [(I.Dims(13, 5, 300, 7, nw), 0.02), (I.Dims(9, 9, 129, 5, nw), 1.0),
         (I.Dims(17, 0, 200, 4, nw), 0.5)])]
    probs[0].wtilde_array[:, ::7] = 1e-8 + 1e-8j
    say(f"[batched] real poles nfreq {nw} schedule {sched}")
    plan = gpp.Plan([p.dims.as_tuple() for p in probs])
    ach, asx = gpp.sigma_batched(plan, [to_device(p) for p in probs])
    torch.cuda.synchronize()
    for k, p in enumerate(probs):
        ref = oracle.sigma_fwd(p)
        assert_parity(ach[k].cpu().numpy(), ref[0], ref[2], f"state {k} achtemp")
        assert_parity(asx[k].cpu().numpy(), ref[1], ref[3], f"state {k} asxtemp")
    plan.close()
