"""trim_memory hands what contexts keep free back to the driver; spaces in use
stay."""
import pytest
import torch

import workloads as W

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

DEV = "cuda:0"


def test_trim_memory():
    import paper_2005_03070_amd as tg
    op = tg.Operator.const_cd((1023, 255), (1.0, 0.0), device=DEV)
    basis = torch.tensor(W.rng(1).standard_normal((48, op.n)), device=DEV)
    space = tg.defl_from_basis(op, basis)
    H = space.basis()[1]
    for _ in range(2):  # about 300 MB each for the space and its workspaces
        tg.defl_from_basis(op, basis)
    torch.cuda.empty_cache()
    before = torch.cuda.mem_get_info()[0]
    tg.trim_memory()
    assert torch.cuda.mem_get_info()[0] >= before + (150 << 20)
    assert (space.basis()[1] == H).all()
    tg.trim_memory()
