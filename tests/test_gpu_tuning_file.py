"""Saved launch shapes of the subspace products: no kernel takes one any more."""
import json

import pytest

from gpu_util import to_dev
from paper_1610_07522_amd import inputs, sky

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("saved", [None, 1, 8, 3])
def test_square_split_of_a_saved_file(tmp_path, saved):
    w = inputs.small_workload("file", 8, 40, 5)
    box = sky.Box(sky.desc_from_workload(w))
    box.init_box(*map(to_dev, inputs.raw_states(w)))
    cache = tmp_path / "tune.json"
    box.autotune(str(cache))
    held = json.loads(cache.read_text())
    assert not any(k.startswith("square_split") for k in held)
    if saved is not None:
        held["square_split/m40"] = saved
        cache.write_text(json.dumps(held))
    t = box.autotune(str(cache))
    assert t["from_cache"] and t["square_split"] == [1, 1]
    assert json.loads(cache.read_text()) == held
