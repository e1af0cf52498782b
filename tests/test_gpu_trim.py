"""trim_memory hands what contexts keep free back to the driver, spaces in use
stay; and a space may be destroyed after its context."""
import ctypes as C

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


def test_a_space_destroyed_after_its_context():
    """The space's memory goes back to the driver."""
    from paper_2005_03070_amd import _lib as L
    lib = L.lib()
    basis = torch.tensor(W.rng(1).standard_normal((48, 1023 * 255)), device=DEV)
    torch.cuda.synchronize()
    ctx, op, space = C.c_void_p(), C.c_void_p(), C.c_void_p()
    L.check(lib.tgdk_ctx_create(C.byref(ctx), 0, None))
    d = L.OpDesc()
    d.dim, d.kind = 2, L.CONST_CD
    d.n[0], d.n[1], d.n[2] = 1023, 255, 1
    d.beta[0] = 1.0
    L.check(lib.tgdk_op_create(ctx, C.byref(d), C.byref(op)))
    L.check(lib.tgdk_defl_from_basis(op, C.c_void_p(basis.data_ptr()), 48, 0, L.F64, C.byref(space)))
    L.check(lib.tgdk_op_destroy(op))
    L.check(lib.tgdk_ctx_destroy(ctx))
    before = torch.cuda.mem_get_info()[0]
    L.check(lib.tgdk_defl_destroy(space))
    assert torch.cuda.mem_get_info()[0] >= before + (48 * 1023 * 255 * 8 >> 1)
