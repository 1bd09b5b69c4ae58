"""Wavefront accumulators at the edges of their segments, against the oracle.

Columns whose product counts stand at, just below and just above every segment
size, formed so that stored B entries cross the rows of a segment, runs of
equal rows cross lanes (up to a whole segment in one run), and A columns
without entries stand between the others. Equal means the same structure and
the same bits: the kernels add in Algorithm 1's order.
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

COUNTS = sorted({c for s in (4, 8, 16, 32, 64, 128, 256, 512, 1024)
                 for c in (s // 2 + 1, s - 1, s, s + 1)} | {1, 2, 3})


def _columns(style, m, seed):
    """(A, B): several columns of B for every count in COUNTS."""
    rng = np.random.default_rng(seed)
    acols, bcols = [], []

    def acol(rows):
        acols.append(np.asarray(rows, np.int64))
        return len(acols) - 1

    empty = acol([])
    for c in COUNTS:
        for rep in range(3):
            if style == "one_entry":  # one A column of c rows
                b = [acol(rng.permutation(np.arange(c) + (m - c if rep else 0)))]
            elif style == "one_row":  # c stored entries, one row: a single run
                b = [acol([(0, m - 1, m // 2)[rep]]) for _ in range(c)]
            else:  # entries of 0 to 9 rows out of few rows: many short runs
                b, left, span = [], c, max(10, c // 3)
                while left:
                    z = min(left, int(rng.integers(1, 10)))
                    b.append(acol(rng.choice(span, z, replace=False) + (m - span if rep else 0)))
                    left -= z
                    if rep == 2 and len(b) % 3 == 0 and len(b) < c // 2:
                        b.append(empty)
            bcols.append(b)
    # an A column stands at most once in a column of B
    used = [np.asarray(list(dict.fromkeys(b)), np.int64) for b in bcols]
    acp = np.concatenate([[0], np.cumsum([len(r) for r in acols])]).astype(np.int32)
    bcp = np.concatenate([[0], np.cumsum([len(b) for b in used])]).astype(np.int32)
    ari = np.concatenate(acols).astype(np.int32)
    bri = np.concatenate(used).astype(np.int32)
    A = gen.CSC(m, len(acols), acp, ari, rng.standard_normal(len(ari)))
    B = gen.CSC(len(acols), len(used), bcp, bri, rng.standard_normal(len(bri)))
    B.val[::7] = -0.0
    return A, B


@pytest.mark.parametrize("m", [1100, 1 << 21], ids=["keys32", "keys64"])
@pytest.mark.parametrize("style", ["one_entry", "one_row", "mixed"])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_segment_edges(style, m, dtype):
    print(f"[case] segment edges {style} m={m} {dtype}", flush=True)
    np_t = np.float64 if dtype == "f64" else np.float32
    A, B = (x.astype(np_t) for x in _columns(style, m, 5))
    ocp, ori, ov = oracle.spgemm(A, B, dtype)
    At, Bt = api.CscTensor.from_host(A), api.CscTensor.from_host(B)
    cp, ri, v = api.matmul(At, Bt).to_host()
    assert_same_structure(cp, ri, ocp, ori, style)
    assert_values_exact(v, ov, style)
    # the one-call product on a kept plan fills at the previous positions
    plan, cpt, rit, vt, nnz = api.multiply(At, Bt)
    for _ in range(2):
        plan, cpt, rit, vt, nnz = api.multiply(At, Bt, plan=plan, out=(cpt, rit, vt))
        torch.cuda.synchronize()
        assert_same_structure(cpt.cpu().numpy(), rit[:nnz].cpu().numpy(), ocp, ori, style)
        assert_values_exact(vt[:nnz].cpu().numpy(), ov, style)
    assert plan.stats()["later_max"] == _depth(A, B)
    plan.close()


def _depth(A, B):
    """Most products adding into one entry of C, less one."""
    deep = 0
    for j in range(B.ncols):
        rows = [A.rowidx[A.colptr[k]:A.colptr[k + 1]]
                for k in B.rowidx[B.colptr[j]:B.colptr[j + 1]]]
        rows = np.concatenate(rows) if rows else np.zeros(0, np.int32)
        if len(rows):
            deep = max(deep, int(np.unique(rows, return_counts=True)[1].max()) - 1)
    return deep


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_row_clusters(dtype):
    """Long columns whose rows stand in clusters of 1 to 14 neighbours, far
    apart: the bucket sort's fullest bucket holds as many keys, up to above the
    limit from which the sorting network takes over; in descending, ascending
    and mixed order, with and without a second product on every row."""
    print(f"[case] row clusters {dtype}", flush=True)
    np_t = np.float64 if dtype == "f64" else np.float32
    rng = np.random.default_rng(9)
    m = 1 << 20
    acols, bcols = [], []
    for size in range(1, 15):
        for total in (300, 512, 700, 1024, 2500):
            starts = np.arange(total // size) * (m // (total // size + 1))
            rows = (starts[:, None] + np.arange(size)).ravel()
            for order in ("down", "up", "mixed"):
                r = rows[::-1] if order == "down" else rows if order == "up" else rng.permutation(rows)
                half = len(r) // 2
                acols += [r[:half], r[half:], r[:half:2]]
                k = len(acols)
                bcols.append([k - 3, k - 2] if order != "mixed" else [k - 1, k - 3, k - 2])
    acp = np.concatenate([[0], np.cumsum([len(r) for r in acols])]).astype(np.int32)
    bcp = np.concatenate([[0], np.cumsum([len(b) for b in bcols])]).astype(np.int32)
    ari = np.concatenate(acols).astype(np.int32)
    bri = np.concatenate(bcols).astype(np.int32)
    A = gen.CSC(m, len(acols), acp, ari, rng.standard_normal(len(ari)).astype(np_t))
    B = gen.CSC(len(acols), len(bcols), bcp, bri, rng.standard_normal(len(bri)).astype(np_t))
    ocp, ori, ov = oracle.spgemm(A, B, dtype)
    cp, ri, v = api.matmul(api.CscTensor.from_host(A), api.CscTensor.from_host(B)).to_host()
    assert_same_structure(cp, ri, ocp, ori, "clusters")
    assert_values_exact(v, ov, "clusters")


@pytest.mark.parametrize("kinds", ["light", "groups", "waves", "light groups", "light waves heavy",
                                   "light groups waves heavy"])
@pytest.mark.parametrize("size", ["one stream", "streams"])
def test_bins_share_launches(kinds, size):
    """Every mix of the kinds of columns that are launched together, with a
    bin's columns just below, at and just above whole work items, below and
    above the product count from which the kinds run on streams of their own;
    a kept plan then takes a B with other counts in every bin."""
    print(f"[case] shared launches {kinds} {size}", flush=True)
    counts = {"light": (4, 8, 16, 32, 64), "groups": (128, 256), "waves": (512, 1024),
              "heavy": (1500, 5000)}
    m = 8192
    rng = np.random.default_rng(11)
    lens = sorted({c // d for cs in counts.values() for c in cs for d in (1, 2)})
    acols = [rng.permutation(m)[:z] for z in lens for _ in range(4)]
    acp = np.concatenate([[0], np.cumsum([len(r) for r in acols])]).astype(np.int32)
    A = gen.CSC(m, len(acols), acp, np.concatenate(acols).astype(np.int32),
                rng.standard_normal(acp[-1]))

    def b_matrix(shift):
        cols = []
        for kind in kinds.split():
            for c in counts[kind]:
                item = 64 if c <= 8 else max(1, 64 * 4 // c)
                fill = 0 if size == "one stream" else (1 << 21) // (c * len(counts[kind]))
                half = 4 * lens.index(c // 2)
                for i in range(item * 2 + shift + fill):
                    # two A columns of c / 2 rows, or one of them
                    a, b = rng.choice(4, 2, replace=False)
                    cols.append([half + a] if i % 9 == 8 and c > 4 else [half + a, half + b])
        cols = [cols[i] for i in rng.permutation(len(cols))]
        bcp = np.concatenate([[0], np.cumsum([len(b) for b in cols])]).astype(np.int32)
        return gen.CSC(len(acols), len(cols), bcp, np.concatenate(cols).astype(np.int32),
                       rng.standard_normal(bcp[-1]))

    At = api.CscTensor.from_host(A)
    plan = out = None
    for shift in (-1, 0, 0, 1):
        B = b_matrix(shift)
        ocp, ori, ov = oracle.spgemm(A, B, "f64")
        plan, *out, nnz = api.multiply(At, api.CscTensor.from_host(B), plan=plan, out=out)
        torch.cuda.synchronize()
        cpt, rit, vt = out
        assert_same_structure(cpt.cpu().numpy(), rit[:nnz].cpu().numpy(), ocp, ori, kinds)
        assert_values_exact(vt[:nnz].cpu().numpy(), ov, kinds)
    plan.close()


@pytest.mark.parametrize("nb", [1, 63, 64, 65, 129, 255, 257, 1030])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_long_columns_in_parts(nb, dtype):
    """Columns of more than 4096 products of nb stored B entries (a part of a
    column takes at least 64 of them), among entries whose A columns are empty
    or hold most of the products, beside columns that are not split."""
    print(f"[case] long columns {nb} {dtype}", flush=True)
    np_t = np.float64 if dtype == "f64" else np.float32
    rng = np.random.default_rng(13)
    m = 9000
    lens = np.full(nb, 5000 // nb + 1)
    lens[rng.permutation(nb)[:nb // 3]] = 0
    lens[nb // 2] = 4097  # the count's bulk, in the middle part
    lens = np.concatenate([lens, [1500, 700, 30]])
    acp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ari = np.concatenate([rng.permutation(m)[:z] for z in lens]).astype(np.int32)
    long = np.arange(nb)
    cols = [long, [nb], long[::-1], [nb, nb + 1, nb + 2], rng.permutation(nb), [nb + 2],
            np.arange(nb + 3)]
    bcp = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32)
    A = gen.CSC(m, len(lens), acp, ari, rng.standard_normal(len(ari)).astype(np_t))
    B = gen.CSC(len(lens), len(cols), bcp, np.concatenate(cols).astype(np.int32),
                rng.standard_normal(bcp[-1]).astype(np_t))
    ocp, ori, ov = oracle.spgemm(A, B, dtype)
    At, Bt = api.CscTensor.from_host(A), api.CscTensor.from_host(B)
    plan, out = None, None
    for _ in range(2):
        plan, *out, nnz = api.multiply(At, Bt, plan=plan, out=out)
        torch.cuda.synchronize()
        assert_same_structure(out[0].cpu().numpy(), out[1][:nnz].cpu().numpy(), ocp, ori, nb)
        assert_values_exact(out[2][:nnz].cpu().numpy(), ov, nb)
    plan.close()
