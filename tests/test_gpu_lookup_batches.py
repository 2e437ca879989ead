"""Lookups on both sides of the sizes at which a lane reads the first entry of
its walk alone (2,048 requests, 64 chunks of a request), in a table with erased
keys and long walks, against the oracle (whole numbers, so exactly)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_35065_amd as kv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("requests", [2047, 2048, 3000])
def test_batches(requests):
    rng = np.random.default_rng(requests)
    live = 4000                                             # of 8,192 positions
    idx = kv.KvIndex(4096)
    keys = rng.integers(0, 2 ** 63, 6000, dtype=np.int64).astype(np.uint64)
    keys[0] = 0
    slots = np.arange(6000, dtype=np.int32)
    idx.insert(keys[:live], slots[:live])
    idx.erase(keys[1000:2000])                              # tombstones on the walks
    idx.insert(keys[live:live + 900], slots[live:live + 900])
    ref = {int(k): int(s) for k, s in zip(keys[:live], slots[:live]) if not 1000 <= s < 2000}
    ref.update({int(k): int(s) for k, s in zip(keys[live:live + 900], slots[live:live + 900])})
    nb = rng.choice([0, 1, 63, 64, 65, 128, 130], requests)
    off = np.concatenate([[0], np.cumsum(nb)]).astype(np.int64)
    present = np.array(sorted(ref), np.uint64)
    bh = rng.choice(present, int(off[-1]))                  # runs of hits ...
    gone = rng.random(int(off[-1])) < 0.02                  # ... that end at erased or never staged keys
    bh[gone] = rng.choice(np.concatenate([keys[1000:2000], keys[live + 900:]]), int(gone.sum()))
    cs = torch.full((int(off[-1]) + 1,), -7, dtype=torch.int32, device="cuda")
    hit = torch.full((requests + 1,), -7, dtype=torch.int32, device="cuda")
    d_off = torch.from_numpy(off).cuda()
    kv.kv_lookup(idx, torch.from_numpy(bh.view(np.int64)).cuda(), d_off, requests, 1, d_off, cs, hit)
    ocs, ohit = oracle.lookup(ref, bh, off, 1)
    assert np.array_equal(cs.cpu().numpy(), np.append(ocs, -7))
    assert np.array_equal(hit.cpu().numpy(), np.append(ohit, -7))
    idx.destroy()
