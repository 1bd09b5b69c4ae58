"""Gradients at the edges of the backward kernels, bit for bit against the oracle.

A columns longer than a chunk of products (512), chunk and wavefront ends
inside and between stored entries, B rows short and long (above 64 entries),
rows and columns without entries; one gradient at a time; and plans whose
allocator refuses the space of the terms, so that dA gathers G itself.
"""
import numpy as np
import pytest

import oracle
from paper_2303_02471_amd import inputs as gen
from helpers import HAVE_GPU

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not HAVE_GPU, reason="needs an MI355X GPU")]

if HAVE_GPU:
    import torch
    from paper_2303_02471_amd import _lib, api


def _csc(rng, nrows, counts):
    cp = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    ri = np.concatenate([rng.permutation(nrows)[:c] for c in counts] + [np.zeros(0, int)])
    return gen.CSC(nrows, len(counts), cp, ri.astype(np.int32), rng.standard_normal(len(ri)))


def _case(name):
    rng = np.random.default_rng(len(name))
    if name == "tiny":
        return _csc(rng, 5, [2, 0, 5]), _csc(rng, 3, [1, 0, 3, 2])
    if name == "long_columns":  # products of a wavefront: several chunks of 512
        return (_csc(rng, 2600, list(rng.choice([0, 1, 7, 511, 512, 513, 1024, 2500], size=90))),
                _csc(rng, 90, list(rng.integers(0, 9, size=60))))
    if name == "exact_chunks":  # 64 entries of 8 products: one chunk exactly
        return _csc(rng, 300, [8] * 50), _csc(rng, 50, [16] * 40)
    if name == "long_rows":  # every B row holds up to 700 entries
        return _csc(rng, 400, list(rng.integers(0, 6, size=12))), _csc(rng, 12, [8] * 700 + [0] * 30)
    return gen.powerlaw(4000, seed=3)


def _check(A, B, need, dtype="f64"):
    np_t = np.float64 if dtype == "f64" else np.float32
    A, B = A.astype(np_t), B.astype(np_t)
    ocp, ori, ov = oracle.spgemm(A, B, dtype)
    G = gen.gradient_values(len(ov), seed=8, dtype=np_t)
    odA, odB = oracle.backward(A, B, ocp, ori, G, dtype)
    At, Bt = api.CscTensor.from_host(A), api.CscTensor.from_host(B)
    C, plan = api.matmul(At, Bt, return_plan=True)
    Gt = torch.from_numpy(G).cuda()
    for _ in range(2):  # builds the view, then runs on it
        dA, dB = api.backward(plan, At.val, Bt.val, C.rowidx, Gt, need_a="a" in need,
                              need_b="b" in need)
        if "a" in need:
            assert np.array_equal(dA.cpu().numpy(), odA), "dA"
        if "b" in need:
            assert np.array_equal(dB.cpu().numpy(), odB), "dB"
    plan.close()


@pytest.mark.parametrize("name", ["tiny", "long_columns", "exact_chunks", "long_rows", "powerlaw"])
@pytest.mark.parametrize("need", ["ab", "a", "b"])
def test_shapes(name, need):
    print(f"[case] backward shapes {name} {need}", flush=True)
    _check(*_case(name), need)


@pytest.mark.parametrize("name", ["long_columns", "long_rows"])
def test_float(name):
    print(f"[case] backward shapes {name} f32", flush=True)
    _check(*_case(name), "ab", "f32")


@pytest.mark.parametrize("name", ["long_columns", "long_rows", "powerlaw"])
def test_without_space_for_the_terms(name):
    print(f"[case] backward without terms {name}", flush=True)
    A, B = _case(name)
    terms = 8 * int(oracle.opcount(A, B).sum())
    refused = []

    def alloc(nbytes, stream, ctx):
        if int(nbytes) == terms:
            refused.append(int(nbytes))
            return None
        return torch.cuda.caching_allocator_alloc(int(nbytes), stream=int(stream or 0))

    def free(ptr, nbytes, stream, ctx):
        torch.cuda.caching_allocator_delete(int(ptr))

    cbs = (_lib.ALLOC_FN(alloc), _lib.FREE_FN(free))
    api.set_allocator(*cbs)
    try:
        _check(A, B, "ab")
        _check(A, B, "a")
    finally:
        api.set_allocator("torch")
    assert refused
