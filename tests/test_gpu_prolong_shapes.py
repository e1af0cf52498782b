"""Prolongation where a wave holds several rows (1 to 31 coarse points: widths of
2 to 32 lanes and their edges), one row (2048 rows and columns together, and
more), and a part of one (fewer), in 2-D and 3-D, with a last group of rows or a
last part that is not full: equal to the oracle's bit for bit."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import transfer as T

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

DEV = "cuda:0"


@pytest.mark.parametrize("cdims", [(nx, 21) for nx in (1, 2, 3, 4, 7, 8, 15, 16, 30, 31, 32, 63, 64)] +
                         [(nx, 2) for nx in (126, 127, 128, 1023, 1024, 4100)] + [(64, 340), (64, 341), (200, 341)] + [(1, 1), (2, 700), (1, 1, 1), (1, 2, 40),
                                                                         (3, 4, 5), (31, 2, 3), (32, 3, 2),
                                                                         (1024, 1, 2)])
def test_prolongation_bits(cdims):
    import paper_2005_03070_amd as tg
    fdims = tuple(2 * d + 1 for d in cdims)
    beta = (0.1,) * len(cdims)
    coarse, fine = tg.Operator.const_cd(cdims, beta, device=DEV), tg.Operator.const_cd(fdims, beta, device=DEV)
    v = W.rng(3).standard_normal((3, coarse.n))
    out = tg.prolongate(coarse, fine, torch.tensor(v, device=DEV)).cpu().numpy()
    for j in range(3):
        assert np.array_equal(out[j], T.prolongate(v[j], cdims))
