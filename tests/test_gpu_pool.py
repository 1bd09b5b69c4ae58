"""Plans that share pooled side streams, events and host buffers, one after the
other and from several threads and streams at once, against the oracle."""
import threading

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


def _equal(C, want, what):
    cp, ri, v = C.to_host()
    assert_same_structure(cp, ri, want[0], want[1], what)
    assert_values_exact(v, want[2], what)


def test_plans_in_turn_and_after_release():
    print("[case] pool: plans in turn", flush=True)
    small, large = gen.uniform_z(300, 3, 1), gen.powerlaw(60000, seed=2)  # 1.5 M products
    want_s, want_l = oracle.spgemm(small, small), oracle.spgemm(*large)
    st = api.CscTensor.from_host(small)
    lt = [api.CscTensor.from_host(x) for x in large]
    for i in range(3):
        _equal(api.matmul(st, st), want_s, "small")
        _equal(api.matmul(*lt), want_l, "large")
        # more header words and upload room than the buffers kept so far
        for c in api.batched_matmul([(st, st)] * (40 * (i + 1))):
            _equal(c, want_s, "batch")
        if i == 1:
            _lib.lib().spgemm_release_pool()


def test_threads_and_streams():
    print("[case] pool: threads and streams", flush=True)
    mats = [gen.powerlaw(50000 + 3000 * i, seed=10 + i) for i in range(4)]
    want = [oracle.spgemm(a, b) for a, b in mats]
    dev = [tuple(api.CscTensor.from_host(x) for x in m) for m in mats]
    torch.cuda.synchronize()
    failed = []

    def work(i):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                for _ in range(6):
                    C = api.matmul(*dev[i])
                    s.synchronize()
                    _equal(C, want[i], f"thread {i}")
        except BaseException as e:  # noqa: BLE001 (reported by the main thread)
            failed.append((i, repr(e)))

    ts = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not failed, failed
