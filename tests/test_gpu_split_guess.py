"""A batch of fewer bits than the last one, large enough that its buckets overflow the
counts made for more bits: it takes the radix passes and the next one of its length
is split.  The path is read from the sort phase's bytes per key (40: split, 24 per
pass plus 24: passes); counts against the oracle."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_shorter_keys_split_again(orc):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2305_05055_amd as cp
    base = orc.build_set(synth.uniform_keys(3000, 7900, bits=40))
    c, expect = cp.CPMA(base), base
    for step, (k, bits, want) in enumerate([(20000, 40, 144), (20000, 40, 40), (1 << 18, 36, 144), (1 << 18, 36, 40),
                                            (1 << 18, 36, 40)]):
        keys = synth.uniform_keys(k, 7910 + step, bits=bits)
        keys[:3] = (1 << bits) - 1, 1, 2  # the bit length, unsorted
        c.stats_select(["sort"])
        expect, added = orc.insert(expect, keys)
        assert c.insert_batch(keys) == added
        per_key = c.stats()["sort"][2] / k
        c.stats_select([])
        assert per_key == want, (step, per_key)
    assert c.size() == len(expect)
    c.close()
