"""Planning kernels at the edges of their tiles, against the oracle.

Column counts around the steps of the tile size and around the number of tiles
up to which the place kernel combines the tiles itself, with columns above
1024 products of every size class at the ends of tiles; batches with more
problems than that many tiles; the column-pointer scan of one workgroup and
just above it.
"""
import numpy as np
import pytest

import oracle
from paper_2303_02471_amd import inputs as gen
from helpers import HAVE_GPU, assert_same_structure, assert_values_exact

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not HAVE_GPU, reason="needs an MI355X GPU")]

if HAVE_GPU:
    import torch
    from paper_2303_02471_amd import api

M = 3000
LENGTHS = [0, 1, 2, 3, 5, 9, 1025, 2049, 2900]


def _a_matrix(rng):
    lens = np.array(LENGTHS * 2)
    rows = np.concatenate([rng.permutation(M)[:z] for z in lens]).astype(np.int32)
    cp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    return gen.CSC(M, len(lens), cp, rows, rng.standard_normal(len(rows)))


def _b_matrix(n, rng, heavy_at):
    """Short columns (0 to 3 entries of the short A columns), and at every
    index of heavy_at one, two or three long A columns (1025 .. 8700 products)."""
    cnt = rng.integers(0, 4, size=n)
    heavy = {int(j): 1 + i % 4 for i, j in enumerate(h for h in heavy_at if 0 <= h < n)}
    for j, c in heavy.items():
        cnt[j] = c
    cp = np.concatenate([[0], np.cumsum(cnt)]).astype(np.int32)
    ri = np.empty(cp[-1], np.int32)
    base = rng.integers(0, 6, size=max(len(ri), 1))  # distinct short columns: base, base + 1, ... mod 6
    pos = np.arange(len(ri)) - np.repeat(cp[:-1], cnt)
    ri[:] = (np.repeat(base[np.minimum(cp[:-1], max(len(ri) - 1, 0))], cnt) + pos) % 6
    for i, (j, c) in enumerate(heavy.items()):
        long = [6, 7, 8, 15, 16, 17]
        ri[cp[j]:cp[j] + c] = [long[(i + q) % 6] for q in range(c)]
    return gen.CSC(len(LENGTHS) * 2, n, cp, ri, rng.standard_normal(len(ri)))


def _check(A, B, what):
    ocp, ori, ov = oracle.spgemm(A, B)
    At, Bt = api.CscTensor.from_host(A), api.CscTensor.from_host(B)
    plan, cp, ri, v, nnz = api.multiply(At, Bt)
    for _ in range(3):  # the first structure, then planned launches
        torch.cuda.synchronize()
        assert_same_structure(cp.cpu().numpy(), ri[:nnz].cpu().numpy(), ocp, ori, what)
        assert_values_exact(v[:nnz].cpu().numpy(), ov, what)
        plan, cp, ri, v, nnz = api.multiply(At, Bt, plan=plan, out=(cp, ri, v))
    s = plan.stats()
    op = oracle.opcount(A, B)
    assert s["total_products"] == int(op.sum()) and s["nnz_c"] == len(ov)
    assert s["cols_empty"] == int((op == 0).sum())
    plan.close()


@pytest.mark.parametrize("n", [1, 7, 8, 9, 8191, 8192, 8193, 16384, 16385, 20000, 655361, 700001])
def test_tile_counts(n):
    print(f"[case] planning tiles n={n}", flush=True)
    rng = np.random.default_rng(n)
    tile = 8
    while tile < 512 and n > 1024 * tile:
        tile *= 2
    edges = [0, n - 1, tile - 1, tile, n // 2, n // 2 // tile * tile, 3 * tile - 1]
    edges += list(rng.integers(0, n, size=30))
    _check(_a_matrix(rng), _b_matrix(n, rng, edges), f"n={n}")


def test_all_columns_heavy():
    print("[case] planning tiles, every column heavy", flush=True)
    rng = np.random.default_rng(3)
    _check(_a_matrix(rng), _b_matrix(300, rng, range(300)), "all heavy")


def test_plan_reused_for_other_column_counts():
    print("[case] planning tiles, one plan over changing shapes", flush=True)
    rng = np.random.default_rng(4)
    A = _a_matrix(rng)
    At = api.CscTensor.from_host(A)
    plan, out = None, None
    for n in (9000, 40, 20000, 40, 9000, 17000):
        B = _b_matrix(n, rng, [0, n - 1])
        ocp, ori, ov = oracle.spgemm(A, B)
        plan, cp, ri, v, nnz = api.multiply(At, api.CscTensor.from_host(B), plan=plan, out=out)
        out = (cp, ri, v)
        torch.cuda.synchronize()
        assert_same_structure(cp.cpu().numpy(), ri[:nnz].cpu().numpy(), ocp, ori, f"n={n}")
        assert_values_exact(v[:nnz].cpu().numpy(), ov, f"n={n}")
    plan.close()


@pytest.mark.parametrize("count", [3, 1400])
def test_batch_tiles(count):
    print(f"[case] planning tiles, batch of {count}", flush=True)
    rng = np.random.default_rng(count)
    A = _a_matrix(rng)
    At = api.CscTensor.from_host(A)
    Bs = [_b_matrix(int(n), rng, [0] if i % 9 == 0 else [])
          for i, n in enumerate(rng.integers(0, 30 if count > 99 else 3000, size=count))]
    pairs = [(At, api.CscTensor.from_host(B)) for B in Bs]
    out = api.batched_matmul(pairs)
    torch.cuda.synchronize()
    for i in range(0, count, max(1, count // 40)):
        ocp, ori, ov = oracle.spgemm(A, Bs[i])
        cp, ri, v = out[i].to_host()
        assert_same_structure(cp, ri, ocp, ori, f"problem {i}")
        assert_values_exact(v, ov, f"problem {i}")
