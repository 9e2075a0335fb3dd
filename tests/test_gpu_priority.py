"""The request order where a thread's requests end: those it keeps, those it reads again."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_12065_amd as ann

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("n,G", [(16, 6), (17, 2), (511, 6), (2048, 6), (2049, 32), (4096, 33), (4097, 6), (6145, 7), (9001, 64),
                                 (2047, 4), (2048, 20), (2049, 21), (4097, 21), (600, 1024)])
def test_priority_requests_held_and_read_again(n, G):
    """Equal levels and equal times throughout, infinite times among them: places are decided by every word of the comparison."""
    gen = np.random.default_rng(n)
    R, C = (gen.integers(lo, hi, n).astype(np.int32) for lo, hi in ((-5, 4), (-100, 8192)))
    W = np.round(gen.random(n) * 60.0, 1)
    Wcur = gen.choice([0.0, -0.0, 1.0, np.nextafter(1.0, 2.0), 1.0 + 2.0 ** -20, -3.5, 1e300, np.inf, -np.inf, np.nan], n)
    level, order = ann.ann_priority_order(torch.from_numpy(R).to(DEV), torch.from_numpy(W).to(DEV), torch.from_numpy(C).to(DEV),
                                          torch.from_numpy(Wcur).to(DEV), G)
    o_level, o_order = oracle.priority_order(R, W, C, Wcur, G)
    assert np.array_equal(level.cpu().numpy(), o_level) and np.array_equal(order.cpu().numpy(), o_order)


@pytest.mark.parametrize("n,G", [(1023, 6), (1024, 21), (1025, 6), (1536, 33), (3071, 21), (3072, 6), (3073, 6), (3073, 64), (2560, 13)])
def test_priority_number_of_requests_held(n, G):
    """Two, four or six requests of a thread are all that there are, or not all."""
    test_priority_requests_held_and_read_again(n, G)
