"""Malformed inputs on plans whose fresh workspace holds arbitrary numbers."""
import numpy as np
import pytest

import oracle
from paper_2303_02471_amd import inputs as gen
from helpers import HAVE_GPU, assert_same_structure, assert_values_exact

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not HAVE_GPU, reason="needs an MI355X GPU")]

if HAVE_GPU:
    import torch
    from paper_2303_02471_amd import _lib, api


@pytest.mark.parametrize("ncols", [7, 700, 60000])
@pytest.mark.parametrize("word", [0, 18, 40, 333, 9000, -1, -40, 2 ** 31 - 1])
def test_workspace_of_any_contents(ncols, word):
    """A row index out of range in the last column (its tile writes no
    accumulator choices): SPGEMM_ERR_CSC whatever the workspace held, and the
    same plan then computes a well-formed product."""
    print(f"[case] malformed, workspace of {word}, {ncols} columns", flush=True)
    held = {}

    def alloc(nbytes, stream, ctx):
        t = torch.full(((int(nbytes) + 3) // 4,), word, dtype=torch.int32, device="cuda")
        held[t.data_ptr()] = t
        return t.data_ptr()

    def free(ptr, nbytes, stream, ctx):
        held.pop(int(ptr), None)

    A = gen.uniform_z(500, 4, seed=1)
    B = gen.uniform_z(ncols, 3, seed=2, nrows=500)
    ri = B.rowidx.copy()
    ri[-1] = 500
    At, Bt = api.CscTensor.from_host(A), api.CscTensor.from_host(B)
    bad = api.CscTensor.from_host(gen.CSC(500, ncols, B.colptr, ri, B.val))
    cbs = (_lib.ALLOC_FN(alloc), _lib.FREE_FN(free))
    api.set_allocator(*cbs)
    try:
        plan = api.Plan()
        with pytest.raises(_lib.SpgemmError) as e:
            api.symbolic(At, bad, torch.float64, plan=plan)
        assert e.value.status == 3
        plan = api.Plan()  # (a first call that fails leaves no plan)
        plan, cp, ri_, v, nnz = api.multiply(At, Bt, plan=plan)
        with pytest.raises(_lib.SpgemmError) as e:
            api.multiply(At, bad, plan=plan, out=(cp, ri_, v))
        assert e.value.status == 3
        plan, cp, ri_, v, nnz = api.multiply(At, Bt, plan=plan, out=(cp, ri_, v))
        torch.cuda.synchronize()
        want = oracle.spgemm(A, B)
        assert_same_structure(cp.cpu().numpy(), ri_[:nnz].cpu().numpy(), want[0], want[1], "after")
        assert_values_exact(v[:nnz].cpu().numpy(), want[2], "after")
        plan.close()
        torch.cuda.synchronize()
    finally:
        api.set_allocator("torch")
    assert not held
