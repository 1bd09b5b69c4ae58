"""Kept plans that meet other structures, options and value types than the ones
their last call left behind, against the oracle."""
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


def _csc(nrows, cols, seed):
    cp = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32)
    ri = np.concatenate([np.asarray(c, np.int32) for c in cols]).astype(np.int32)
    return gen.CSC(nrows, len(cols), cp, ri, np.random.default_rng(seed).uniform(-1, 1, len(ri)))


def _kept(A, Bs, what):
    """One-call products A x B of every B in turn on one plan and its arrays."""
    At = api.CscTensor.from_host(A)
    plan, out = None, None
    for step, B in enumerate(Bs):
        Bt = api.CscTensor.from_host(B)
        plan, cp, ri, v, nnz = api.multiply(At, Bt, plan=plan, out=out)
        out = (cp, ri, v)
        torch.cuda.synchronize()
        want = oracle.spgemm(A, B)
        assert nnz == int(want[0][-1]), f"{what}, step {step}"
        assert_same_structure(cp.cpu().numpy(), ri[:nnz].cpu().numpy(), want[0], want[1],
                              f"{what}, step {step}")
        assert_values_exact(v[:nnz].cpu().numpy(), want[2], f"{what}, step {step}")
    plan.close()


def test_columns_without_products_now():
    """Products and stored entries as many as before, every column that has
    products as long as its old place, and a column that had some has none."""
    print("[case] kept plan: a column loses its products", flush=True)
    A = _csc(3, [[0, 1, 2], [0, 1, 2]], 1)
    B1, B2 = (_csc(2, c, 2) for c in ([[0], [1], [0, 1], []], [[], [0, 1], [0, 1], []]))
    _kept(A, (B1, B1, B2, B2, B1), "empty")


def test_heavy_column_in_a_longer_place():
    """A heavy column that is shorter than the place it now stands in, with the
    window counts of the column that was heavy before."""
    print("[case] kept plan: heavy and light columns exchanged", flush=True)
    rng = np.random.default_rng(3)
    rows = rng.permutation(4000)[:40]
    A = _csc(4000, [rows[:20]] * 60 + [rows[20:]], 4)
    heavy, two, one = list(range(60)), [0, 60], [0, 1]  # 1200 products, 20 rows; 40, 20 of 40
    B1, B2 = _csc(61, [heavy, two], 5), _csc(61, [one, heavy], 5)
    _kept(A, (B1, B1, B2, B2, B1), "heavy")


def test_windows_that_no_launch_has_counted():
    """Many windows of few products, then few windows of more (the scratch is
    laid out anew), then as many products in more windows than the second call
    counted but no more than the first."""
    print("[case] kept plan: more windows than were counted", flush=True)
    rng = np.random.default_rng(7)
    A = gen.uniform_z(5000, 25, seed=8, nrows=4000)

    def B(*entries):  # entries of the first columns of 100
        cols = [rng.permutation(5000)[:n] for n in entries] + [[]] * (100 - len(entries))
        return _csc(5000, cols, 9)

    B2, B3 = B(5000, 41), B(2581, *[41] * 60)
    assert 25 * B2.nnz == 25 * B3.nnz
    _kept(A, (B(*[41] * 100), B2, B2, B3, B3), "windows")


def test_options_and_types_change_on_one_plan():
    """Every accumulator choice after every other one, and both value types, on
    one plan with columns of every size class."""
    print("[case] kept plan: options and types change", flush=True)
    A, B = gen.powerlaw(20000, seed=6)
    opts = [{}, {"radix_esc": True}, {}, {"lane_hash": True}, {"t_block": -1}, {"lane_blocked": True},
            {"radix_esc": True}, {"t_esc": 32}, {"t_block": -1}]
    plan, out = None, {"f64": None, "f32": None}
    for step in range(2 * len(opts)):
        kw, dt = opts[step // 2], ("f64", "f32")[(step + step // 2) % 2]
        np_t = np.float64 if dt == "f64" else np.float32
        a, b = A.astype(np_t), B.astype(np_t)
        want = oracle.spgemm(a, b, dt)
        plan, cp, ri, v, nnz = api.multiply(api.CscTensor.from_host(a), api.CscTensor.from_host(b),
                                            opts=api.options(**kw), plan=plan, out=out[dt])
        out[dt] = (cp, ri, v)
        torch.cuda.synchronize()
        what = f"step {step} {kw} {dt}"
        assert_same_structure(cp.cpu().numpy(), ri[:nnz].cpu().numpy(), want[0], want[1], what)
        assert_values_exact(v[:nnz].cpu().numpy(), want[2], what)
    plan.close()


def test_batched_values_on_two_streams():
    """New value and output arrays on another stream right behind the last call:
    each call's kernels meet their own problem table."""
    print("[case] kept plan: batched numeric on two streams", flush=True)
    mats = [(gen.uniform_z(30000, 12, seed=20 + i), gen.uniform_z(30000, 12, seed=30 + i))
            for i in range(2)]
    dev = [tuple(api.CscTensor.from_host(x) for x in m) for m in mats]
    plan, cps, nnzs = api.batched_symbolic(dev)
    sets = []
    for scale in (1.0, 2.0, 4.0, 8.0):
        pairs = [(api.CscTensor(a.nrows, a.ncols, a.colptr, a.rowidx, a.val * scale), b) for a, b in dev]
        sets.append((scale, pairs, [torch.zeros(z, dtype=torch.int32, device="cuda") for z in nnzs],
                     [torch.zeros(z, dtype=torch.float64, device="cuda") for z in nnzs]))
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for i, (_, pairs, ris, vs) in enumerate(sets):
        api.batched_numeric(plan, pairs, ris, vs, stream=streams[i % 2])
    torch.cuda.synchronize()
    for p, (A, B) in enumerate(mats):
        want = oracle.spgemm(A, B)
        for scale, _, ris, vs in sets:
            assert_same_structure(cps[p].cpu().numpy(), ris[p].cpu().numpy(), want[0], want[1], f"{scale}")
            assert_values_exact(vs[p].cpu().numpy(), scale * want[2], f"{scale}")
    plan.close()
