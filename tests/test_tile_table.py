"""The shipped tile table: from d = 8 on the batch's families (oscillatory, product
peak, Gaussian) have factored kernels, with one lane per region; an entry that asks
for several lanes there would take the chain-form kernel instead."""
import json
import os

from paper_2511_01573_amd import autotune


def test_no_entry_gives_up_the_factored_kernel():
    assert os.path.exists(autotune.DEFAULT_TABLE)
    with open(autotune.DEFAULT_TABLE) as fh:
        table = json.load(fh)
    assert len(table) == 24
    several = {k for k, v in table.items() if v["d"] >= 8 and v["lanes_per_region"] != 1}
    assert not several
