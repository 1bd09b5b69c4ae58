"""Gradients in both forms (two passes over the products; one launch with a thread
per stored entry), bit for bit against the oracle: a plan's first call takes
the two passes, later ones the form that its sizes and longest lists make the
faster. Lists of 0 to 9 terms around the one-launch form's 4 terms at a time."""
import numpy as np
import pytest

import oracle
from paper_2303_02471_amd import inputs as gen
from helpers import HAVE_GPU

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not HAVE_GPU, reason="needs an MI355X GPU")]

if HAVE_GPU:
    import torch
    from paper_2303_02471_amd import api


def _random_lists(seed):
    """Columns of 0 to 9 entries in A and B, rows of B as uneven."""
    rng = np.random.default_rng(seed)

    def csc(nrows, ncols):
        cols = [rng.permutation(nrows)[:rng.integers(0, 10)] for _ in range(ncols)]
        cp = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32)
        ri = np.concatenate(cols).astype(np.int32)
        return gen.CSC(nrows, ncols, cp, ri, rng.standard_normal(len(ri)))
    return csc(700, 257), csc(257, 511)


CASES = {"short lists": lambda: _random_lists(1),            # one launch
         "one entry": lambda: (gen.uniform_z(3, 1, seed=1), gen.uniform_z(3, 1, seed=2)),
         "uniform": lambda: (gen.uniform_z(2500, 40, seed=3), gen.uniform_z(2500, 40, seed=4)),  # two
         "power law": lambda: gen.powerlaw(15000, seed=5)}   # two: long lists


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_forms(name, dtype):
    print(f"[case] backward forms {name} {dtype}", flush=True)
    np_t = np.float64 if dtype == "f64" else np.float32
    A, B = (x.astype(np_t) for x in CASES[name]())
    ocp, ori, ov = oracle.spgemm(A, B, dtype)
    At, Bt = api.CscTensor.from_host(A), api.CscTensor.from_host(B)
    Cm, plan = api.matmul(At, Bt, return_plan=True)
    for call, need in enumerate(("ab", "ab", "a", "b", "ab")):
        G = gen.gradient_values(len(ov), seed=call, dtype=np_t)
        want = oracle.backward(A, B, ocp, ori, G, dtype)
        got = api.backward(plan, At.val, Bt.val, Cm.rowidx, torch.from_numpy(G).cuda(),
                           need_a="a" in need, need_b="b" in need)
        torch.cuda.synchronize()
        for x, w, n in zip(got, want, "ab"):
            if n in need:
                assert np.array_equal(x.cpu().numpy(), w), f"d{n.upper()}, call {call}"
    plan.close()


def _setup(A, B, grads):
    ocp, ori, ov = oracle.spgemm(A, B)
    At, Bt = api.CscTensor.from_host(A), api.CscTensor.from_host(B)
    Cm, plan = api.matmul(At, Bt, return_plan=True)
    Gs = [gen.gradient_values(len(ov), seed=40 + i, dtype=np.float64) for i in range(grads)]
    want = [oracle.backward(A, B, ocp, ori, G) for G in Gs]
    dev = [torch.from_numpy(G).cuda() for G in Gs]
    api.backward(plan, At.val, Bt.val, Cm.rowidx, dev[0])  # builds the view
    torch.cuda.synchronize()
    return At, Bt, Cm, plan, dev, want


def _equal(got, want, what):
    for x, w, n in zip(got, want, "AB"):
        assert np.array_equal(x.cpu().numpy(), w), f"{what}: d{n}"


def test_two_streams():
    """Gradients of one plan on two streams without a wait between them."""
    print("[case] backward on two streams", flush=True)
    At, Bt, Cm, plan, dev, want = _setup(*gen.powerlaw(60000, seed=7), 6)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for s in streams:
        s.wait_stream(torch.cuda.current_stream())
    outs = [(torch.zeros_like(At.val), torch.zeros_like(Bt.val)) for _ in dev]
    torch.cuda.synchronize()
    for i, (G, out) in enumerate(zip(dev, outs)):
        api.backward(plan, At.val, Bt.val, Cm.rowidx, G, out=out, stream=streams[i % 2])
    torch.cuda.synchronize()
    for i, out in enumerate(outs):
        _equal(out, want[i], f"call {i}")
    plan.close()


def test_replays_beside_other_gradients():
    """Replays of gradients captured twice (with the terms' space, and without
    any left) on streams of their own while eager ones of the same plan run on
    another."""
    print("[case] captured backward beside eager backward", flush=True)
    At, Bt, Cm, plan, dev, want = _setup(*gen.powerlaw(60000, seed=8), 6)
    outs = [(torch.zeros_like(At.val), torch.zeros_like(Bt.val)) for _ in dev]
    streams, other = [torch.cuda.Stream(), torch.cuda.Stream()], torch.cuda.Stream()
    graphs = [torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()]
    for g, s, G, out in zip(graphs, streams, dev, outs):
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            with torch.cuda.graph(g, stream=s):
                api.backward(plan, At.val, Bt.val, Cm.rowidx, G, out=out)
    torch.cuda.synchronize()
    for r in range(3):
        for o in outs:
            o[0].zero_(), o[1].zero_()
        torch.cuda.synchronize()
        for i in range(2, len(dev)):
            for g, s in zip(graphs, streams):
                with torch.cuda.stream(s):
                    g.replay()
            api.backward(plan, At.val, Bt.val, Cm.rowidx, dev[i], out=outs[i], stream=other)
        torch.cuda.synchronize()
        for i, o in enumerate(outs):
            _equal(o, want[i], f"round {r}, gradient {i}")
    plan.close()
