"""The prefix hash where its chain changes shape: around whole tiles (256
blocks), groups of 64 and steps of 8, alone and in a batch, against the
oracle (whole numbers, so exactly)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_35065_amd as kv

pytestmark = pytest.mark.gpu

BLOCKS = [1, 7, 8, 9, 56, 57, 63, 64, 65, 72, 127, 128, 255, 256, 257, 264, 319, 320, 511, 512, 513, 520, 767, 768,
          769, 1024, 1031]


def _run(lengths, seed):
    rng = np.random.default_rng(len(lengths))
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    toks = rng.integers(0, 32000, int(off[-1])).astype(np.int32)
    blk = oracle.block_offsets(off)
    out = torch.full((int(blk[-1]) + 8,), -1, dtype=torch.int64, device="cuda")   # eight words past the end stay
    kv.kv_hash_prefix(torch.from_numpy(toks).cuda(), torch.from_numpy(off).cuda(), len(lengths), seed,
                      torch.from_numpy(blk).cuda(), out)
    got = out.cpu().numpy()
    assert np.array_equal(got[:-8].view(np.uint64), oracle.hash_prefix(toks, off, seed))
    assert (got[-8:] == -1).all()


@pytest.mark.parametrize("blocks", BLOCKS)
def test_one_request(blocks):
    _run([blocks * 16 + blocks % 3], 9)


def test_batch():
    _run([b * 16 for b in BLOCKS] * 40, 2 ** 64 - 1)


def test_short_requests():
    # every length from nothing to past a group of 64, whose last blocks run as single steps, some tokens over
    _run([b * 16 + b % 16 for b in range(0, 75)] * 8, 3)
